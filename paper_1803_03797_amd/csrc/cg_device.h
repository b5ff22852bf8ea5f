// cg_device.h - device code the kernel sources share: a lane's row of a
// vector, the wavefront exchanges, the operators at a point, the scalar step
// between two passes (the recurrences of Algorithms 1 and 2) and the
// deterministic reductions.
#pragma once
#include <math.h>

#include "cg_internal.h"

namespace cgk {

// ------------------------------------------------------------- lane rows --

template <typename T, int CPL>
struct Row {
  T e[CPL];
};

template <typename T, int CPL>
__device__ __forceinline__ Row<T, CPL> zrow() {
  Row<T, CPL> v;
#pragma unroll
  for (int k = 0; k < CPL; ++k) v.e[k] = T(0);
  return v;
}

template <typename T, int CPL>
__device__ __forceinline__ Row<T, CPL> ldrow(const T* p) {
  Row<T, CPL> v;
  if constexpr (sizeof(T) == 8) {
#pragma unroll
    for (int k = 0; k < CPL; k += 2) {
      double2 t = *reinterpret_cast<const double2*>(p + k);
      v.e[k] = t.x;
      v.e[k + 1] = t.y;
    }
  } else {
#pragma unroll
    for (int k = 0; k < CPL; k += 4) {
      float4 t = *reinterpret_cast<const float4*>(p + k);
      v.e[k] = t.x;
      v.e[k + 1] = t.y;
      v.e[k + 2] = t.z;
      v.e[k + 3] = t.w;
    }
  }
  return v;
}

// Stores the first `valid` elements (valid >= CPL: the whole row segment).
template <typename T, int CPL>
__device__ __forceinline__ void strow(T* p, const Row<T, CPL>& v, int valid) {
  if (valid >= CPL) {
    if constexpr (sizeof(T) == 8) {
#pragma unroll
      for (int k = 0; k < CPL; k += 2)
        *reinterpret_cast<double2*>(p + k) = make_double2(v.e[k], v.e[k + 1]);
    } else {
#pragma unroll
      for (int k = 0; k < CPL; k += 4)
        *reinterpret_cast<float4*>(p + k) =
            make_float4(v.e[k], v.e[k + 1], v.e[k + 2], v.e[k + 3]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < CPL; ++k)
      if (k < valid) p[k] = v.e[k];
  }
}

// ---------------------------------------------------- wavefront exchange --

constexpr int kDppWaveShr1 = 0x138;  // lane l receives lane l-1 (lane 0 keeps `old`)
constexpr int kDppWaveShl1 = 0x130;  // lane l receives lane l+1 (lane 63 keeps `old`)

template <int CTRL>
__device__ __forceinline__ double dpp(double v, double old) {
  int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, 0xf, 0xf,
                                       false);
  int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, 0xf, 0xf,
                                       false);
  return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v, float old) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL,
                                                    0xf, 0xf, false));
}

// West and east neighbours of every element of a lane's row segment.  eW is
// the value left of the tile (used by lane 0), eE the value right of it
// (used by lane 63).  Must be called with the whole wavefront active.
template <typename T, int CPL>
__device__ __forceinline__ void west_east(const Row<T, CPL>& v, T eW, T eE, Row<T, CPL>& W,
                                          Row<T, CPL>& E) {
  W.e[0] = dpp<kDppWaveShr1>(v.e[CPL - 1], eW);
  E.e[CPL - 1] = dpp<kDppWaveShl1>(v.e[0], eE);
#pragma unroll
  for (int k = 1; k < CPL; ++k) W.e[k] = v.e[k - 1];
#pragma unroll
  for (int k = 0; k < CPL - 1; ++k) E.e[k] = v.e[k + 1];
}

// (A u) at one point: (((4 uC - uW) - uE) - uS) - uN, S = row j-1, N = row j+1.
template <typename T>
__device__ __forceinline__ T st5(T c, T w, T e, T s, T n) {
  return (((T(4) * c - w) - e) - s) - n;
}

// The same value in one operation less, for kernels that the arithmetic bounds:
// 4 c is exact, so the fma rounds as the product and the subtraction do.
template <typename T>
__device__ __forceinline__ T st5_fma(T c, T w, T e, T s, T n) {
  return ((fma(T(4), c, -w) - e) - s) - n;
}

// The operator at one point, selected by OP:
//   0: the 5-point stencil;
//   1: the 7-point one in 3D, (((((6 uC - uW) - uE) - uS) - uN) - uB) - uT,
//      B = plane l-1, T = plane l+1;
//   2: the variable-coefficient 5-point one with face conductivities kw, ke,
//      ks, kn: d = ((kw + ke) + ks) + kn, then (((d uC - kw uW) - ke uE) -
//      ks uS) - kn uN, each product rounded before its subtraction.
template <int OP, typename T>
__device__ __forceinline__ T stn(T c, T w, T e, T s, T n, T b, T t, T kw, T ke, T ks, T kn) {
  if constexpr (OP == 1) {
    return (((((T(6) * c - w) - e) - s) - n) - b) - t;
  } else if constexpr (OP == 2) {
    const T d = ((kw + ke) + ks) + kn;
    const T pc = d * c, pw = kw * w, pe = ke * e, ps = ks * s, pn = kn * n;
    return (((pc - pw) - pe) - ps) - pn;
  } else {
    return st5(c, w, e, s, n);
  }
}

// The four face conductivities of a lane's cells on one row.
template <typename T, int CPL>
struct Kc {
  Row<T, CPL> w, e, s, n;
};

// The operator at column k of a lane's row from the walker's rows.
template <int OP, typename T, int CPL, class KC>
__device__ __forceinline__ T op_at(const Row<T, CPL>& S, const Row<T, CPL>& C,
                                   const Row<T, CPL>& N, const Row<T, CPL>& W,
                                   const Row<T, CPL>& E, const Row<T, CPL>& B,
                                   const Row<T, CPL>& U, const KC& kc, int k) {
  if constexpr (OP == 2) {
    return stn<2>(C.e[k], W.e[k], E.e[k], S.e[k], N.e[k], T(0), T(0), kc.w.e[k], kc.e.e[k],
                  kc.s.e[k], kc.n.e[k]);
  } else {
    return stn<OP>(C.e[k], W.e[k], E.e[k], S.e[k], N.e[k], B.e[k], U.e[k], T(0), T(0), T(0),
                   T(0));
  }
}

// Reads a State every lane needs with the same value into scalar registers
// (readfirstlane), so the solve's scalars do not hold vector registers (which
// the compiler would otherwise spill across the prologue's barriers).
__device__ __forceinline__ State load_state_uniform(const State* p) {
  static_assert(sizeof(State) % 16 == 0, "State is loaded as uint4");
  constexpr int N = sizeof(State) / 4;
  uint32_t u[N];
  const uint4* q = reinterpret_cast<const uint4*>(p);
#pragma unroll
  for (int i = 0; i < N / 4; ++i) {
    const uint4 v = q[i];
    u[4 * i + 0] = __builtin_amdgcn_readfirstlane(v.x);
    u[4 * i + 1] = __builtin_amdgcn_readfirstlane(v.y);
    u[4 * i + 2] = __builtin_amdgcn_readfirstlane(v.z);
    u[4 * i + 3] = __builtin_amdgcn_readfirstlane(v.w);
  }
  State s;
  __builtin_memcpy(&s, u, sizeof(State));
  return s;
}

// The same for a State held in registers whose fields are uniform (all
// threads computed them from the same sums).
__device__ __forceinline__ State uniform_state(const State& in) {
  constexpr int N = sizeof(State) / 4;
  uint32_t u[N];
  __builtin_memcpy(u, &in, sizeof(State));
#pragma unroll
  for (int i = 0; i < N; ++i) u[i] = __builtin_amdgcn_readfirstlane(u[i]);
  State s;
  __builtin_memcpy(&s, u, sizeof(State));
  return s;
}

__device__ __forceinline__ double uniform(double v) {
  const int lo = __builtin_amdgcn_readfirstlane(__double2loint(v));
  const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(v));
  return __hiloint2double(hi, lo);
}

// DPP controls that are xor permutations inside 16-lane rows.
constexpr int kDppXor8 = 0x128;  // row_ror:8: lane l of a 16-lane row gets lane l ^ 8
constexpr int kDppXor2 = 0x4E;   // quad_perm [2,3,0,1]: lane l gets lane l ^ 2
constexpr int kDppXor1 = 0xB1;   // quad_perm [1,0,3,2]: lane l gets lane l ^ 1

constexpr int kDppHalfMirror = 0x141;  // lane l of 8 gets lane l ^ 7
constexpr int kDppXor3 = 0x1B;         // quad_perm [3,2,1,0]: lane l gets lane l ^ 3

// 64-bit values (double or int64_t) across lanes without LDS: gfx950's lane
// swaps exchange halves of 32 and of 16 lanes, DPP permutes within 16.
template <typename T>
__device__ __forceinline__ T from_halves(unsigned hi, unsigned lo) {
  return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T swap_add32(T v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return from_halves<T>(h[0], l[0]) + from_halves<T>(h[1], l[1]);
}
template <typename T>
__device__ __forceinline__ T swap_add16(T v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)b, hi = (unsigned)(b >> 32);
  const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  return from_halves<T>(h[0], l[0]) + from_halves<T>(h[1], l[1]);
}

// A lane permutation that every lane takes part in.
template <int CTRL, typename T>
__device__ __forceinline__ T perm(T v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return from_halves<T>((unsigned)hi, (unsigned)lo);
}

// The sum over 16 lanes: an xor butterfly, stages 8, 4, 2, 1.
template <typename T>
__device__ __forceinline__ T row_sum_valu(T v) {
  v = v + perm<kDppXor8>(v);
  v = v + perm<kDppXor3>(perm<kDppHalfMirror>(v));  // l ^ 7 ^ 3 = l ^ 4
  v = v + perm<kDppXor2>(v);
  v = v + perm<kDppXor1>(v);
  return v;
}

// The sum over the wavefront: stages 32, 16, ..., 1 (every lane adds its xor
// partner's value; addition commutes).
template <typename T>
__device__ __forceinline__ T wave_sum_valu(T v) {
  return row_sum_valu(swap_add16(swap_add32(v)));
}

__device__ __forceinline__ bool uniform_flag(bool b) {
  return __builtin_amdgcn_readfirstlane((int)b) != 0;
}

// ------------------------------------------------------- tile geometry --

struct Strip {
  int tx, lane, wave;
  int c;       // first column of this lane
  int ct;      // first column of the tile
  int j0, j1;  // rows of this wavefront's strip, j0, j0 + js, ... < j1; empty
               // when j0 >= j1
  int js;      // row step: 1, or the rows of a plane (3D z-march)
  int y;       // 3D: the wavefront's in-plane row (may lie past the plane)
  int z0, z1;  // 3D: the tile's planes [z0, z1), the same for its wavefronts
};

// 2D: tile t = ty * ntx + tx of 4 wavefronts x rows rows; wavefront w walks
// rows ty * th + w * rows + [0, rows).  3D (g.plane > 0, the z-march): tile
// t = (tz * nty + ty) * ntx + tx of 4 consecutive in-plane rows (one per
// wavefront: y = ty * 4 + w) by rows planes; wavefront w walks its row y
// through planes tz * rows + [0, rows), one plane (g.plane stored rows) per
// step.
template <int CPL>
__device__ __forceinline__ Strip strip_of(const Geo& g, int t) {
  Strip s;
  s.tx = t % g.ntx;
  const int ty = t / g.ntx;
  s.lane = threadIdx.x & (kWave - 1);
  s.wave = (threadIdx.x >> 6) & (kWavesPerTile - 1);
  s.ct = s.tx * (kWave * CPL);
  s.c = s.ct + s.lane * CPL;
  if (g.plane > 0) {
    const int pl = g.plane, nz = g.ny / pl;
    const int y = (ty % g.nty) * kWavesPerTile + s.wave;
    const int z0 = (ty / g.nty) * g.rows, z1 = min(z0 + g.rows, nz);
    s.js = pl;
    s.y = y;
    s.z0 = z0;
    s.z1 = z1;
    s.j0 = s.j1 = 0;
    if (y < pl) {
      s.j0 = z0 * pl + y;
      s.j1 = z1 * pl + y;
    }
    return s;
  }
  s.js = 1;
  s.y = s.z0 = s.z1 = 0;
  s.j0 = ty * g.th + s.wave * g.rows;
  s.j1 = min(s.j0 + g.rows, g.ny);
  return s;
}

// Values just outside the tile on one row (zero outside the grid: the pad
// columns are zero, and there is no tile beyond the last one).
template <typename T, int CPL>
__device__ __forceinline__ void edges(const T* row, const Strip& s, const Geo& g, T& eW, T& eE) {
  eW = T(0);
  eE = T(0);
  if (s.lane == 0 && s.tx > 0) eW = row[s.ct - 1];
  if (s.lane == kWave - 1 && s.tx + 1 < g.ntx) eE = row[s.ct + kWave * CPL];
}

// ---------------------------------------------------------- scalar step --


__device__ __forceinline__ int stop_code(double gamma, double thr, int k, int maxit, double tol) {
  if (!isfinite(gamma)) return ST_BREAKDOWN;
  if (gamma <= thr) return ST_OK;
  if (k >= maxit) return tol == 0.0 ? ST_OK : ST_NOT_CONVERGED;
  return ST_RUNNING;
}

// Applies the scalar recurrences that sit between the previous pass and this
// one.  `sum` holds the cross-tile sums of the previous pass's partials.
// Returns true when this pass's body must run.
template <int KIND>
__device__ __forceinline__ bool transition(State& s, const double* sum, Sc& sc) {
  sc.al = 0.0;
  sc.be = 0.0;
  sc.first = 0;
  sc.xu = 0;
  sc.inv = 0.0;
  sc.alp = 0.0;
  if constexpr (KIND == K_PCGX) {
    return transition<K_PCG>(s, sum, sc);
  } else if constexpr (KIND == K_CG2X) {
    return transition<K_CG2>(s, sum, sc);
  } else if constexpr (KIND == K_CG2FX) {
    return transition<K_CG2F>(s, sum, sc);
  } else if constexpr (KIND == K_APPLY || KIND == K_DOT || KIND == K_RESID) {
    return true;
  } else if constexpr (KIND == K_RRQ || KIND == K_RRZ) {
    return s.status == ST_RUNNING;
  } else if constexpr (KIND == K_INIT_R) {
    return s.status == ST_RUNNING;
  } else if constexpr (KIND == K_INIT_W) {
    if (s.status != ST_RUNNING) return false;
    s.bb = sum[1];
    s.thr = (s.tol * s.tol) * s.bb;
    s.flags &= ~F_BB_PENDING;
    if (s.bb == 0.0) s.status = ST_ZERO_RHS;
    return s.status == ST_RUNNING;
  } else if constexpr (KIND == K_INIT_WU) {
    return s.status == ST_RUNNING;
  } else if constexpr (KIND == K_CHEBW) {
    // Preconditioned pipelined CG: gamma = (r,u), delta = (w,u) and the stop
    // test on (r,r); first pass alpha = gamma/delta, later beta =
    // gamma/gamma_old, alpha = 1/(delta/gamma - beta/alpha_old).  gamma is
    // kept in gamma0 (State::gamma holds (r,r), the residual reported).
    if (s.status != ST_RUNNING) return false;
    const double gu = sum[0], du = sum[1], rr = sum[2];
    int st = stop_code(rr, s.thr, s.k, s.maxit, s.tol);
    double al = 0.0, be = 0.0;
    if (st == ST_RUNNING) {
      if (s.k == 0) {
        if (!(du > 0.0) || !isfinite(du)) st = ST_BREAKDOWN;
        else al = gu / du;
      } else {
        be = gu / s.gamma0;
        const double den = du / gu - be / s.alpha;
        if (!(den > 0.0) || !isfinite(den)) st = ST_BREAKDOWN;
        else al = 1.0 / den;
      }
    }
    s.gamma = rr;
    s.gamma0 = gu;
    s.delta = du;
    s.status = st;
    if (st != ST_RUNNING) return false;
    s.alpha = al;
    s.beta = be;
    s.k += 1;
    return true;
  } else if constexpr (KIND == K_PPCG) {
    // the scalars of this iteration were set by the Chebyshev pass before it
    if (s.status != ST_RUNNING) return false;
    sc.al = s.alpha;
    sc.be = s.beta;
    sc.first = s.k == 1;
    return true;
  } else if constexpr (KIND == K_PCG) {
    // Algorithm 2: gamma = (r,r), delta = (w,r); first pass alpha = gamma/delta,
    // later beta = gamma/gamma_old, alpha = 1/(delta/gamma - beta/alpha_old).
    if (s.status != ST_RUNNING) return false;
    const double gamma = sum[0], delta = sum[1];
    int st = stop_code(gamma, s.thr, s.k, s.maxit, s.tol);
    double al = 0.0, be = 0.0;
    if (st == ST_RUNNING) {
      if (s.k == 0) {
        if (!(delta > 0.0) || !isfinite(delta)) st = ST_BREAKDOWN;
        else al = gamma / delta;
        sc.first = 1;
      } else {
        be = gamma / s.gamma;
        const double den = delta / gamma - be / s.alpha;
        if (!(den > 0.0) || !isfinite(den)) st = ST_BREAKDOWN;
        else al = 1.0 / den;
      }
    }
    s.gamma = gamma;
    s.delta = delta;
    s.status = st;
    if (st != ST_RUNNING) return false;
    s.alpha = al;
    s.beta = be;
    s.k += 1;
    sc.al = al;
    sc.be = be;
    return true;
  } else if constexpr (KIND == K_CHEB) {
    // Preconditioned CG: the stop test on gamma = (r,r) of the current
    // residual (from the initial residual pass or classic pass 2, which also
    // brings (b,b) the first time), before z = M^-1 r is formed.
    if (s.status != ST_RUNNING) return false;
    const double gamma = sum[0];
    if (s.flags & F_BB_PENDING) {
      s.bb = sum[1];
      s.thr = (s.tol * s.tol) * s.bb;
      s.flags &= ~F_BB_PENDING;
      if (s.bb == 0.0) {
        s.status = ST_ZERO_RHS;
        return false;
      }
    }
    const int st = stop_code(gamma, s.thr, s.k, s.maxit, s.tol);
    s.gamma = gamma;
    s.status = st;
    return st == ST_RUNNING;
  } else if constexpr (KIND == K_CG1) {
    // Algorithm 1: beta = (r,r)_new / (r,r)_old, then p = r + beta p.
    // Preconditioned: the one slot is rho = (r,z) from the Chebyshev pass
    // (which already made the stop test); beta = rho_new / rho_old with rho
    // kept in delta, then p = z + beta p.
    if (s.status != ST_RUNNING) return false;
    const double gamma = sum[0];
    if (s.flags & F_PRECOND) {
      const double rho = sum[0];
      double be = 0.0;
      if (!(rho > 0.0) || !isfinite(rho)) {
        s.status = ST_BREAKDOWN;
        return false;
      }
      if (s.k == 0) sc.first = 1;
      else be = rho / s.delta;
      s.delta = rho;
      s.beta = be;
      sc.be = be;
      return true;
    }
    if (s.flags & F_BB_PENDING) {
      s.bb = sum[1];
      s.thr = (s.tol * s.tol) * s.bb;
      s.flags &= ~F_BB_PENDING;
      if (s.bb == 0.0) {
        s.status = ST_ZERO_RHS;
        return false;
      }
    }
    const int st = stop_code(gamma, s.thr, s.k, s.maxit, s.tol);
    double be = 0.0;
    if (s.k == 0) sc.first = 1;
    else be = gamma / s.gamma;
    s.gamma = gamma;
    s.delta = gamma;  // alpha's numerator for pass 2
    s.status = st;
    if (st != ST_RUNNING) return false;
    s.beta = be;
    sc.be = be;
    return true;
  } else if constexpr (KIND == K_CG2) {
    // Algorithm 1: alpha = (r,r) / (p, A p).
    if (s.status != ST_RUNNING) return false;
    const double pi = sum[0];
    if (!(pi > 0.0) || !isfinite(pi)) {
      s.status = ST_BREAKDOWN;
      return false;
    }
    // delta holds alpha's numerator: rho = (r,z) preconditioned, else (r,r)
    // (one field read unconditionally: a select between two fields of the
    // state would make the compiler address it through scratch memory)
    s.alpha = s.delta / pi;
    s.k += 1;
    sc.al = s.alpha;
    return true;
  } else if constexpr (KIND == K_REF_SCALE) {
    // Outer refinement step: test the true FP64 residual, then scale it.
    if (s.status != ST_RUNNING) return false;
    const double g = sum[0];
    if (s.flags & F_BB_PENDING) {
      s.bb = sum[1];
      s.thr = (s.tol * s.tol) * s.bb;
      s.flags &= ~F_BB_PENDING;
      if (s.bb == 0.0) {
        s.status = ST_ZERO_RHS;
        return false;
      }
    }
    s.res2 = g;
    int st = ST_RUNNING;
    if (!isfinite(g)) st = ST_BREAKDOWN;
    else if (g <= s.thr) st = ST_OK;
    else if (s.k >= s.maxit) st = ST_NOT_CONVERGED;
    s.status = st;
    if (st != ST_RUNNING) return false;
    s.scale = sqrt(g);
    s.kin = 0;
    sc.inv = 1.0 / s.scale;
    return true;
  } else if constexpr (KIND == K_CHEBF) {
    // Preconditioned inner solve: the inner stop test on gamma = (r, r) of
    // the inner residual (the scale pass or pass 2 before this one), before
    // z = M^-1 r is formed; the threshold as in the unpreconditioned one.
    if (s.status != ST_RUNNING) return false;
    const double gamma = sum[0];
    if (s.kin == 0) {
      const double e = fmax(s.inner_tol, (0.5 * s.tol) * (sqrt(s.bb) / s.scale));
      s.gamma0 = gamma;
      s.thr_in = (e * e) * gamma;
    }
    s.gamma = gamma;
    if (!isfinite(gamma) || gamma <= s.thr_in || s.k >= s.maxit) {
      s.status = ST_INNER_DONE;
      return false;
    }
    return true;
  } else if constexpr (KIND == K_CG1F) {
    if (s.status != ST_RUNNING) return false;
    if (s.flags & F_PRECOND) {
      // the one slot is rho = (r, z) from the Chebyshev pass (which made the
      // stop test); beta = rho / rho_old with rho kept in delta, p = z + beta p
      const double rho = sum[0];
      if (!(rho > 0.0) || !isfinite(rho)) {
        s.status = ST_INNER_DONE;
        return false;
      }
      double be = 0.0;
      if (s.kin == 0) sc.first = 1;
      else be = rho / s.delta;
      s.delta = rho;
      s.beta = be;
      sc.be = be;
      return true;
    }
    const double gamma = sum[0];
    double be = 0.0;
    if (s.kin == 0) {
      // inner stop: relative residual e = max(inner_tol, (tol/2) ||b|| / s),
      // no further than the outer tolerance needs (s = ||b - A x||)
      const double e = fmax(s.inner_tol, (0.5 * s.tol) * (sqrt(s.bb) / s.scale));
      s.gamma0 = gamma;
      s.thr_in = (e * e) * gamma;
      sc.first = 1;
    } else {
      be = gamma / s.gamma;
    }
    s.gamma = gamma;
    s.delta = gamma;  // alpha's numerator for pass 2
    if (!isfinite(gamma) || gamma <= s.thr_in || s.k >= s.maxit) {
      s.status = ST_INNER_DONE;
      return false;
    }
    s.beta = be;
    sc.be = be;
    return true;
  } else if constexpr (KIND == K_CG2F) {
    if (s.status != ST_RUNNING) return false;
    const double pi = sum[0];
    if (!(pi > 0.0) || !isfinite(pi)) {
      s.status = ST_INNER_DONE;
      return false;
    }
    // delta: rho = (r, z) preconditioned, else (r, r)
    s.alpha = s.delta / pi;
    s.k += 1;
    s.kin += 1;
    sc.al = s.alpha;
    return true;
  } else if constexpr (KIND == K_REF_UPDATE) {
    if (s.status != ST_INNER_DONE) return false;
    if (s.kin == 0) {
      s.status = ST_BREAKDOWN;
      return false;
    }
    s.status = ST_RUNNING;
    s.outer += 1;
    sc.al = s.scale;
    return true;
  }
  return false;
}

template <int KIND>
constexpr int ndots_in() {  // partial slots the prologue consumes
  return (KIND == K_PCG || KIND == K_PCGX || KIND == K_INIT_W || KIND == K_CG1 ||
          KIND == K_REF_SCALE)
             ? 2
         : (KIND == K_CG2 || KIND == K_CG2X || KIND == K_CG1F || KIND == K_CG2F ||
            KIND == K_CG2FX || KIND == K_CHEBF)
             ? 1
             : 0;
}

template <int KIND>
constexpr int ndots_out() {  // partial slots the body produces
  return (KIND == K_INIT_WU || KIND == K_PPCG) ? 3
         : (KIND == K_INIT_R || KIND == K_INIT_W || KIND == K_PCG || KIND == K_PCGX ||
            KIND == K_RESID)
             ? 2
         : (KIND == K_CG1 || KIND == K_CG2 || KIND == K_CG2X || KIND == K_REF_SCALE ||
            KIND == K_CG1F || KIND == K_CG2F || KIND == K_CG2FX || KIND == K_DOT)
             ? 1
             : 0;
}

// The passes whose solution update is deferred (see cg_internal.h): FP64 CG
// (x, counted by k) and the FP32 inner solve (d, counted by kin).
template <int KIND>
constexpr bool defers_x() {
  return KIND == K_PCG || KIND == K_PCGX || KIND == K_CG1 || KIND == K_CG2 || KIND == K_CG2X ||
         KIND == K_CG1F || KIND == K_CG2F || KIND == K_CG2FX || KIND == K_CHEB ||
         KIND == K_CHEBF;
}

template <int KIND>
constexpr bool inner_kind() {
  return KIND == K_CG1F || KIND == K_CG2F || KIND == K_CG2FX || KIND == K_CHEBF;
}

// transition<KIND> plus the deferred-x bookkeeping: sc.xu when this pass ends
// an even iteration (sc.alp = the previous iteration's alpha), and `flush`
// when this pass stops a running solve whose last iteration was odd (then
// sc.alp = that iteration's alpha, whose update is still pending).
template <int KIND>
__device__ __forceinline__ bool transition_x(State& s, const double* sum, Sc& sc, bool& flush) {
  const bool was_running = s.status == ST_RUNNING;
  const double alpha_before = s.alpha;
  const bool run = transition<KIND>(s, sum, sc);
  flush = false;
  if constexpr (defers_x<KIND>()) {
    const int k = inner_kind<KIND>() ? s.kin : s.k;
    if (run && KIND != K_CG1 && KIND != K_CG1F && KIND != K_CHEB && KIND != K_CHEBF &&
        !(k & 1)) {
      sc.xu = 1;
      sc.alp = alpha_before;
    }
    if (was_running && s.status != ST_RUNNING && (k & 1)) {
      flush = true;
      sc.alp = s.alpha;
    }
  }
  return run;
}

// A barrier that orders LDS only: global stores in flight (the exchange words)
// are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ------------------------------------------------------------- reductions --

// Cross-tile stage: the 256 threads of a tile group sum part[d*T + k] for
// k = tid, tid+256, ... in order, butterfly within each wavefront, then add
// the four wavefront values in order.  Every thread of the group receives
// the sums.  `lds` holds 4*D doubles for this group.
// Every work-group of a pass waits for this before it starts: with one load at
// a time that was about 10 us of each pipelined pass of 4096 x 4096 (two sums of
// 4096 tiles): 264.6 -> 254.0 us an iteration with kLoads, and
// 27.1 -> 24.7 us at 1024 x 1024, preconditioned by s = 2 steps.
template <int D>
__device__ __forceinline__ void cross_tile_sum(const double* part, int T, double* out,
                                               double* lds) {
  const int tid = threadIdx.x & (kGroup - 1), lane = tid & (kWave - 1), wave = tid >> 6;
  // kLoads at a time (one after the other, each would wait for the last: the
  // partials come from the other XCDs, past this one's L2)
  constexpr int kLoads = D == 1 ? 8 : 4;
  double v[D] = {};
  for (int k0 = tid; k0 < T; k0 += kLoads * kGroup) {
    double t[D][kLoads];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int u = 0; u < kLoads; ++u)
        t[d][u] = part[(size_t)d * T + min(k0 + u * kGroup, T - 1)];
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int u = 0; u < kLoads; ++u)
        v[d] = v[d] + (k0 + u * kGroup < T ? t[d][u] : 0.0);  // never -0, so + 0 is no change
  }
#pragma unroll
  for (int d = 0; d < D; ++d) v[d] = wave_sum_valu(v[d]);
  if (lane == 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) lds[wave * D + d] = v[d];
  }
  __syncthreads();
#pragma unroll
  for (int d = 0; d < D; ++d) {
    double t = lds[d];
#pragma unroll
    for (int w = 1; w < kWavesPerTile; ++w) t = t + lds[w * D + d];
    out[d] = t;
  }
  __syncthreads();
}

// Per-tile partials: butterfly each lane value, add wavefronts in order, and
// let the group's first thread store part[d*T + t].  `lds` holds 2*4*D
// doubles for this group (double-buffered by `par` so one barrier suffices).
template <int D>
__device__ __forceinline__ void tile_partial(const double* lv, double* part, int T, int t,
                                             double* lds, int par) {
  const int tid = threadIdx.x & (kGroup - 1), lane = tid & (kWave - 1), wave = tid >> 6;
  double* L = lds + par * kWavesPerTile * D;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const double v = wave_sum_valu(lv[d]);
    if (lane == 0) L[wave * D + d] = v;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      double s = L[d];
#pragma unroll
      for (int w = 1; w < kWavesPerTile; ++w) s = s + L[w * D + d];
      part[(size_t)d * T + t] = s;
    }
  }
}

template <int CPL>
__device__ __forceinline__ double fold(const double (&acc)[CPL]) {
  double v = acc[0];
#pragma unroll
  for (int k = 1; k < CPL; ++k) v = v + acc[k];
  return v;
}

}  // namespace cgk
