// cg_onchip.hip - small solves: the whole solve in one work-group with every
// vector on chip.
//
// Threads are laid out in rows of nx + 1: thread t owns column c = t mod
// (nx + 1) and the ROWS rows of segment t div (nx + 1) (rows past ny are held
// as zero); the last thread of each row (c == nx) and the threads past the
// last segment own nothing and hold zeros, so the west neighbour of column 0
// and the east neighbour of column nx - 1 read as zero without a test.  ROWS
// is the least of 2, 5, 10, 20 that keeps the grid within kRrThreads threads:
// few rows a thread mean more wavefronts side by side on a small grid (33 x 17
// has one wavefront at 20 rows, five at two).  Along a column the stencil's
// south / north neighbours are the thread's own registers; west / east
// neighbours come from the adjacent lanes by DPP.  What crosses a thread's
// boundary (the first and last element of every segment, the whole segment of
// lanes 0 and 63 of each wavefront) goes through LDS, together with the
// wavefront sums of the dot products, with one barrier per exchange and the
// LDS buffers double-buffered by phase parity.  Classic CG exchanges r alone:
// a thread keeps the direction of its surroundings and forms the new one from
// their r.  Pipelined CG of 20 rows keeps x in LDS (six vectors of 20 rows do
// not fit the register file); everything else is in registers.
//
// Rows outside the grid hold exact zeros through every update (the stencil
// result is forced to zero there, and every other update maps zeros to +0),
// so the dot products accumulate them without a test: fma(0, 0, acc) == acc.
//
// Dot products follow the column-segment order: fma per thread over its rows
// in ascending order, xor butterfly, wavefronts in order.  Every vector update
// is the same expression as in the pass bodies and every scalar one that of
// the transitions.
//
// Bound by instruction issue in one compute unit (20 rows: about 100 cycles a
// row and wavefront, two wavefronts to a SIMD) and by the dependent chain of a
// sum, a barrier and two or three divisions (few rows: about 1.3 us an iteration
// whatever the grid).  us per iteration, classic / pipelined, against 20 rows a
// thread for every grid, LDS butterflies and the transition's full scalar code
// on every pass:
//   33 x 17    3.8 / 3.7 -> 1.3 / 1.3   (2 rows)
//   40 x 40    3.7 / 3.6 -> 1.5 / 1.5   (5 rows)
//   64 x 64    4.2 / 4.2 -> 1.8 / 2.0   (10 rows)
//   100 x 100  4.3 / 4.3 -> 2.7 / 3.4   (20 rows)
#include "cg_device.h"
#include "cg_internal.h"

namespace cgk {

namespace {

constexpr int kRrWaves = kRrThreads / kWave;

template <int ROWS>
struct RrXchg {  // one exchanged vector
  double first[kRrThreads];  // element 0 of each thread's segment
  double last[kRrThreads];   // element ROWS - 1
  // segments of lanes 0 and 63 of wavefront w at [w + 1]; [0] stays zero (the
  // west neighbour of thread 0)
  double edge[kRrWaves + 1][2][ROWS];
};

template <int ROWS, bool PIPE>
struct RrLds {
  RrXchg<ROWS> x[2];              // by phase parity
  double tot[2][kRrWaves][2];     // wavefront sums, by phase parity (zero for
                                  // wavefronts that are not there)
  double xs[PIPE && ROWS > 10 ? ROWS : 1][kRrThreads];  // pipelined: the iterate x
};

// The iterate of a pipelined solve: in registers, or in LDS where the five
// other vectors leave no room for it.
template <int ROWS>
struct RrIterate {
  static constexpr bool kLds = ROWS > 10;
  double v[kLds ? 1 : ROWS];
  double (*m)[kRrThreads];
  int t;
  __device__ __forceinline__ double get(int e) const { return kLds ? m[e][t] : v[e]; }
  __device__ __forceinline__ void set(int e, double a) {
    if constexpr (kLds) m[e][t] = a;
    else v[e] = a;
  }
};

struct RrSeg {
  int t, lane, wave, nw;
  int stride;         // threads per row of segments (nx + 1)
  int nv;             // rows of the segment inside the grid (0: idle thread)
  bool south, north;  // the segment below / above exists
  size_t off;         // element offset of the segment's first row
  int pitch;
};

template <int ROWS>
__device__ __forceinline__ RrSeg rr_seg(const Geo& g) {
  RrSeg s;
  s.t = threadIdx.x;
  s.lane = s.t & (kWave - 1);
  s.wave = __builtin_amdgcn_readfirstlane(s.t >> 6);
  s.nw = blockDim.x >> 6;
  s.stride = g.nx + 1;
  const int nseg = (g.ny + ROWS - 1) / ROWS;
  const int c = s.t % s.stride, sg = s.t / s.stride;
  const bool act = sg < nseg && c < g.nx;
  s.nv = act ? min(ROWS, g.ny - sg * ROWS) : 0;
  s.south = act && sg > 0;
  s.north = act && sg + 1 < nseg;
  s.pitch = g.pitch;
  s.off = act ? (size_t)sg * ROWS * g.pitch + c : 0;
  return s;
}

// Zeroes what is read but never written: the edge entry of thread 0's west
// neighbour and the sums of absent wavefronts.
template <int ROWS, bool PIPE>
__device__ __forceinline__ void rr_clear(RrLds<ROWS, PIPE>& L) {
  const int t = threadIdx.x;
  if (t < 2 * ROWS) L.x[0].edge[0][t / ROWS][t % ROWS] = L.x[1].edge[0][t / ROWS][t % ROWS] = 0.0;
  if (t < 2 * kRrWaves * 2) (&L.tot[0][0][0])[t] = 0.0;
}

// The segment's addresses are recomputed at every use (the empty asm hides
// the offset from common-subexpression elimination), so the addresses of the
// first load are not kept in registers across the whole solve.
template <int ROWS>
__device__ __forceinline__ void rr_load(const double* G, const RrSeg& s, double (&v)[ROWS]) {
  size_t off = s.off;
  asm volatile("" : "+v"(off));
#pragma unroll
  for (int e = 0; e < ROWS; ++e) v[e] = G && e < s.nv ? G[off + (size_t)e * s.pitch] : 0.0;
}

template <int ROWS>
__device__ __forceinline__ void rr_store(double* G, const RrSeg& s, const double (&v)[ROWS]) {
  size_t off = s.off;
  asm volatile("" : "+v"(off));
#pragma unroll
  for (int e = 0; e < ROWS; ++e)
    if (e < s.nv) G[off + (size_t)e * s.pitch] = v[e];
}

template <int ROWS>
__device__ __forceinline__ void rr_publish(const double (&v)[ROWS], const RrSeg& s,
                                           RrXchg<ROWS>& X) {
  X.first[s.t] = v[0];
  X.last[s.t] = v[ROWS - 1];
  if (s.lane == 0 || s.lane == kWave - 1) {
    double* d = X.edge[s.wave + 1][s.lane == 0 ? 0 : 1];
#pragma unroll
    for (int e = 0; e < ROWS; ++e) d[e] = v[e];
  }
}

// What a thread's segment borders on, of one vector: south of element 0 and
// north of element ROWS - 1, and of every element the wavefront's west (lanes
// 0-31; lane 0 uses it) or east (lanes 32-63; lane 63) neighbour, held in
// registers or read from LDS where it is used.
template <int ROWS>
struct RrHalo {
  double S, N, e[ROWS];
};

struct RrBorder {
  double S, N;
  const double* e;
};

template <int ROWS>
__device__ __forceinline__ RrBorder rr_border(const RrSeg& s, const RrXchg<ROWS>& X) {
  RrBorder h;
  const int ts = s.south ? s.t - s.stride : s.t, tn = s.north ? s.t + s.stride : s.t;
  const double S = X.last[ts], N = X.first[tn];
  h.S = s.south ? S : 0.0;
  h.N = s.north ? N : 0.0;
  // west: lane 63 of the previous wavefront (the zero entry for wavefront 0);
  // east: lane 0 of the next (for the last wavefront an entry nobody uses)
  h.e = s.lane < kWave / 2 ? X.edge[s.wave][1] : X.edge[min(s.wave + 2, s.nw)][0];
  return h;
}

// (A v) at element e of the segment; zero for rows outside the grid.  vs is
// v[e - 1] as it was before any update of this pass (the caller may have
// overwritten v[e - 1] already); unused for e == 0.  The zero is a select or a
// branch (SEL): us per iteration of 64 x 64 and 100 x 100, pipelined 1.97 and
// 3.37 with selects, 2.19 and 3.69 with branches; classic 1.89 and 2.78, 1.85
// and 2.71.
template <int ROWS, bool SEL, class Halo>
__device__ __forceinline__ double rr_st5(const double (&v)[ROWS], double vs, const RrSeg& s,
                                         const Halo& h, int e) {
  const double edge = h.e[e];
  const double w = dpp<kDppWaveShr1>(v[e], edge);   // lane 0 keeps its west edge
  const double ea = dpp<kDppWaveShl1>(v[e], edge);  // lane 63 keeps its east edge
  const double so = e > 0 ? vs : h.S;
  const double no = e + 1 < ROWS ? v[e + 1] : h.N;
  if constexpr (SEL) {
    const double a = st5_fma(v[e], w, ea, so, no);
    return e < s.nv ? a : 0.0;
  }
  return e < s.nv ? st5_fma(v[e], w, ea, so, no) : 0.0;
}

template <int D>
__device__ __forceinline__ void rr_publish_sums(const double* acc, const RrSeg& s,
                                                double (*tot)[2]) {
  double v[D];
#pragma unroll
  for (int d = 0; d < D; ++d) v[d] = wave_sum_valu(acc[d]);
  if (s.lane == 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) tot[s.wave][d] = v[d];
  }
}

// Sums of the wavefront totals in wavefront order (absent ones add zero).
template <int D>
__device__ __forceinline__ void rr_read_sums(const double (*tot)[2], double* sum) {
  double2 t[kRrWaves];
#pragma unroll
  for (int w = 0; w < kRrWaves; ++w) t[w] = *reinterpret_cast<const double2*>(tot[w]);
  double v0 = t[0].x, v1 = t[0].y;
#pragma unroll
  for (int w = 1; w < kRrWaves; ++w) {
    v0 = v0 + t[w].x;
    v1 = v1 + t[w].y;
  }
  sum[0] = uniform(v0);
  if (D > 1) sum[1] = uniform(v1);
}

// r = b - A x of the published x, with its sums (r,r) and (b,b).
template <int ROWS>
__device__ __forceinline__ void rr_residual(const double* B, const RrSeg& s,
                                            const double (&x)[ROWS], const RrXchg<ROWS>& X,
                                            double (&r)[ROWS], double* acc) {
  double b[ROWS];
  rr_load<ROWS>(B, s, b);
  const RrBorder h = rr_border<ROWS>(s, X);
  acc[0] = acc[1] = 0.0;
#pragma unroll
  for (int e = 0; e < ROWS; ++e) {
    r[e] = b[e] - rr_st5<ROWS, false>(x, e > 0 ? x[e - 1] : 0.0, s, h, e);
    acc[0] = fma(r[e], r[e], acc[0]);
    acc[1] = fma(b[e], b[e], acc[1]);
  }
}

// The true residual of the final iterate: res2 = (t,t), t = b - A x.
template <int ROWS, bool PIPE>
__device__ __forceinline__ void rr_final(const RrArgs& a, const RrSeg& s, State& st,
                                         const double (&x)[ROWS], RrLds<ROWS, PIPE>& L,
                                         int par) {
  rr_publish<ROWS>(x, s, L.x[par]);
  lds_barrier();
  double t[ROWS], acc[2], sum[2];
  rr_residual<ROWS>(a.b, s, x, L.x[par], t, acc);
  rr_publish_sums<1>(acc, s, L.tot[par ^ 1]);
  lds_barrier();
  rr_read_sums<1>(L.tot[par ^ 1], sum);
  st.res2 = sum[0];
}

// Pipelined CG (Algorithm 2) on one grid, x in LDS: one sum per iteration.
// The scalars of an iteration are formed here, with the operations of
// transition<K_PCG>, as long as nothing ends the solve; the first iteration, a
// stop and a breakdown go through it.
template <int ROWS>
__device__ __forceinline__ void rr_solve_pcg(const RrArgs& a, State& st, char* raw) {
  using Lds = RrLds<ROWS, true>;
  Lds& L = *reinterpret_cast<Lds*>(raw);
  const RrSeg s = rr_seg<ROWS>(a.g);
  double r[ROWS], w[ROWS], p[ROWS], q[ROWS], z[ROWS];
  Sc sc;
  int par = 0;
  double sum[2] = {0.0, 0.0}, acc[2];
  RrIterate<ROWS> xi;
  xi.m = L.xs;
  xi.t = s.t;
  rr_clear(L);
  {
    double x[ROWS];
    rr_load<ROWS>(a.x0, s, x);
#pragma unroll
    for (int e = 0; e < ROWS; ++e) xi.set(e, x[e]);
    rr_publish<ROWS>(x, s, L.x[par]);
    __syncthreads();
    transition<K_INIT_R>(st, sum, sc);
    rr_residual<ROWS>(a.b, s, x, L.x[par], r, acc);
    par ^= 1;
    rr_publish<ROWS>(r, s, L.x[par]);
    rr_publish_sums<2>(acc, s, L.tot[par]);
    lds_barrier();
  }
  rr_read_sums<2>(L.tot[par], sum);
  if (uniform_flag(transition<K_INIT_W>(st, sum, sc))) {
    // w = A r; slots (r,r), (w,r)
    const RrBorder h0 = rr_border<ROWS>(s, L.x[par]);
    acc[0] = acc[1] = 0.0;
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      w[e] = rr_st5<ROWS, false>(r, e > 0 ? r[e - 1] : 0.0, s, h0, e);
      acc[0] = fma(r[e], r[e], acc[0]);
      acc[1] = fma(w[e], r[e], acc[1]);
      // z = A w, q = w, p = r on the first iteration: beta is 0, and 0 * -0 + v
      // is v bit for bit
      z[e] = q[e] = p[e] = -0.0;
    }
    par ^= 1;
    rr_publish<ROWS>(w, s, L.x[par]);
    rr_publish_sums<2>(acc, s, L.tot[par]);
    lds_barrier();
    rr_read_sums<2>(L.tot[par], sum);
    bool go = uniform_flag(transition<K_PCG>(st, sum, sc));
    st = uniform_state(st);
    double gamma = st.gamma, alpha = st.alpha, beta = st.beta;
    const double thr = st.thr;
    int k = st.k;
    const int maxit = st.maxit;
    while (go) {
      const double al = alpha, be = beta, nal = -alpha;
      const RrBorder h = rr_border<ROWS>(s, L.x[par]);
      acc[0] = acc[1] = 0.0;
      double wprev = 0.0;  // w[e - 1] of this pass (w is updated in place)
#pragma unroll
      for (int e = 0; e < ROWS; ++e) {
        const double nv = rr_st5<ROWS, true>(w, wprev, s, h, e);
        wprev = w[e];
        z[e] = fma(be, z[e], nv);
        q[e] = fma(be, q[e], w[e]);
        p[e] = fma(be, p[e], r[e]);
        xi.set(e, fma(al, p[e], xi.get(e)));
        r[e] = fma(nal, q[e], r[e]);
        w[e] = fma(nal, z[e], w[e]);
        acc[0] = fma(r[e], r[e], acc[0]);
        acc[1] = fma(w[e], r[e], acc[1]);
        // Two rows at a time: left to itself the compiler puts w and the sums of
        // all rows off to the end and keeps a second z and r until then, which
        // at 20 rows is 56 registers spilled on every pass.
        if (e % 2 == 1)
          asm volatile("" : "+v"(w[e]), "+v"(w[e - 1]), "+v"(acc[0]), "+v"(acc[1]));
      }
      par ^= 1;
      rr_publish<ROWS>(w, s, L.x[par]);
      rr_publish_sums<2>(acc, s, L.tot[par]);
      lds_barrier();
      rr_read_sums<2>(L.tot[par], sum);
      const double be1 = sum[0] / gamma;
      const double den = sum[1] / sum[0] - be1 / alpha;
      if (sum[0] > thr && sum[0] < __builtin_huge_val() && k < maxit && den > 0.0 &&
          den < __builtin_huge_val()) {
        beta = be1;
        alpha = 1.0 / den;
        gamma = sum[0];
        k += 1;
      } else {
        st.gamma = gamma;
        st.alpha = alpha;
        st.beta = beta;
        st.k = k;
        go = uniform_flag(transition<K_PCG>(st, sum, sc));
        st = uniform_state(st);
        gamma = st.gamma;
        alpha = st.alpha;
        beta = st.beta;
        k = st.k;
      }
    }
  }
  double x[ROWS];
#pragma unroll
  for (int e = 0; e < ROWS; ++e) x[e] = xi.get(e);
  if (st.status != ST_ZERO_RHS) rr_final<ROWS, true>(a, s, st, x, L, par ^ 1);
  rr_store<ROWS>(a.x, s, x);
}

// Classic CG (Algorithm 1) on one grid, every vector in registers: two sums
// per iteration.  Scalars as above.
template <int ROWS>
__device__ __forceinline__ void rr_solve_cg(const RrArgs& a, State& st, char* raw) {
  using Lds = RrLds<ROWS, false>;
  Lds& L = *reinterpret_cast<Lds*>(raw);
  const RrSeg s = rr_seg<ROWS>(a.g);
  double x[ROWS], r[ROWS], p[ROWS], sv[ROWS];
  Sc sc;
  int par = 0;
  double sum[2] = {0.0, 0.0}, acc[2];
  rr_clear(L);
  rr_load<ROWS>(a.x0, s, x);
  rr_publish<ROWS>(x, s, L.x[par]);
  __syncthreads();
  transition<K_INIT_R>(st, sum, sc);
  rr_residual<ROWS>(a.b, s, x, L.x[par], r, acc);
  par ^= 1;
  rr_publish<ROWS>(r, s, L.x[par]);
  rr_publish_sums<2>(acc, s, L.tot[par]);
  lds_barrier();
  rr_read_sums<2>(L.tot[par], sum);
  bool go = uniform_flag(transition<K_CG1>(st, sum, sc));
  st = uniform_state(st);
  double gamma = st.gamma, alpha = st.alpha, beta = st.beta;
  const double thr = st.thr;
  int k = st.k;
  const int maxit = st.maxit;
  RrHalo<ROWS> ph;  // the direction around the segment
  ph.S = ph.N = -0.0;
#pragma unroll
  for (int e = 0; e < ROWS; ++e) ph.e[e] = p[e] = -0.0;  // first: p = r (see above)
  while (go) {
    const double be = beta;
    const RrBorder h = rr_border<ROWS>(s, L.x[par]);
    ph.S = fma(be, ph.S, h.S);
    ph.N = fma(be, ph.N, h.N);
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      ph.e[e] = fma(be, ph.e[e], h.e[e]);
      p[e] = fma(be, p[e], r[e]);
    }
    acc[0] = 0.0;
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      sv[e] = rr_st5<ROWS, false>(p, e > 0 ? p[e - 1] : 0.0, s, ph, e);
      acc[0] = fma(p[e], sv[e], acc[0]);
    }
    par ^= 1;
    rr_publish_sums<1>(acc, s, L.tot[par]);
    lds_barrier();
    rr_read_sums<1>(L.tot[par], sum);
    if (!(sum[0] > 0.0 && sum[0] < __builtin_huge_val())) {
      st.gamma = st.delta = gamma;
      st.alpha = alpha;
      st.beta = beta;
      st.k = k;
      (void)transition<K_CG2>(st, sum, sc);  // a breakdown
      break;
    }
    alpha = gamma / sum[0];
    k += 1;
    const double al = alpha, nal = -alpha;
    acc[0] = 0.0;
#pragma unroll
    for (int e = 0; e < ROWS; ++e) {
      r[e] = fma(nal, sv[e], r[e]);
      acc[0] = fma(r[e], r[e], acc[0]);
    }
    par ^= 1;
    rr_publish<ROWS>(r, s, L.x[par]);
    rr_publish_sums<1>(acc, s, L.tot[par]);
#pragma unroll
    for (int e = 0; e < ROWS; ++e) x[e] = fma(al, p[e], x[e]);
    lds_barrier();
    rr_read_sums<1>(L.tot[par], sum);
    if (!(sum[0] > thr && sum[0] < __builtin_huge_val() && k < maxit)) {
      st.gamma = st.delta = gamma;
      st.alpha = alpha;
      st.beta = beta;
      st.k = k;
      go = uniform_flag(transition<K_CG1>(st, sum, sc));
      st = uniform_state(st);
    }
    beta = sum[0] / gamma;
    gamma = sum[0];
  }
  if (st.status != ST_ZERO_RHS) rr_final<ROWS, false>(a, s, st, x, L, par ^ 1);
  rr_store<ROWS>(a.x, s, x);
}

template <int ROWS>
constexpr size_t rr_lds(int variant) {
  return variant ? sizeof(RrLds<ROWS, true>) : sizeof(RrLds<ROWS, false>);
}

template <int VARIANT, int ROWS>
__device__ __forceinline__ void rr_solve(const RrArgs& a, State& st, char* raw) {
  if constexpr (VARIANT == 1) rr_solve_pcg<ROWS>(a, st, raw);
  else rr_solve_cg<ROWS>(a, st, raw);
}

template <int VARIANT, int ROWS>
__global__ __launch_bounds__(kRrThreads) void k_solve_rr(RrArgs a) {
  __shared__ __attribute__((aligned(16))) char raw[rr_lds<ROWS>(VARIANT)];
  State st = uniform_state(a.s0);
  rr_solve<VARIANT, ROWS>(a, st, raw);
  if (threadIdx.x == 0) *a.out = st;
}

// The forms of k_solve_rr_many, each a function of its own (side by side in
// one they would share a register allocation).
typedef __attribute__((address_space(3))) char* LdsBytes;

template <int VARIANT, int ROWS>
__device__ __attribute__((noinline)) void rr_call(const Slot* S, LdsBytes lds) {
  RrArgs a = {};
  a.g = S->g;
  a.b = S->b;
  a.x0 = S->x;
  a.x = S->x;
  State st = load_state_uniform(S->S[0]);
  rr_solve<VARIANT, ROWS>(a, st, (char*)lds);
  st.kind = K_DONE;
  if (threadIdx.x == 0) {
    *S->S[0] = st;
    *S->S[1] = st;
  }
}

// Many small solves, one per work-group: work-group i solves the resident
// solve in slot idx[i] (initial state in S[0]) and leaves its final state,
// marked done for the step engine, in both S[0] and S[1].  A wider work-group
// than the solve needs only adds idle wavefronts, whose zero sums leave every
// dot product unchanged.
__global__ __launch_bounds__(kRrThreads) void k_solve_rr_many(const Slot* slots,
                                                              const int* idx) {
  __shared__ __attribute__((aligned(16))) char raw[rr_lds<kRrRows>(1)];
  const Slot* S = slots + __builtin_amdgcn_readfirstlane(idx[blockIdx.x]);
  const int form = __builtin_amdgcn_readfirstlane(rr_rows(S->g.nx, S->g.ny) * 2 + S->variant);
  switch (form) {
    case 4: return rr_call<0, 2>(S, (LdsBytes)raw);
    case 5: return rr_call<1, 2>(S, (LdsBytes)raw);
    case 10: return rr_call<0, 5>(S, (LdsBytes)raw);
    case 11: return rr_call<1, 5>(S, (LdsBytes)raw);
    case 20: return rr_call<0, 10>(S, (LdsBytes)raw);
    case 21: return rr_call<1, 10>(S, (LdsBytes)raw);
    case 40: return rr_call<0, 20>(S, (LdsBytes)raw);
    case 41: return rr_call<1, 20>(S, (LdsBytes)raw);
  }
}

template <int VARIANT>
hipError_t launch_v(const RrArgs& a, int rows, int threads, hipStream_t st) {
  switch (rows) {
    case 2: hipLaunchKernelGGL((k_solve_rr<VARIANT, 2>), dim3(1), dim3(threads), 0, st, a); break;
    case 5: hipLaunchKernelGGL((k_solve_rr<VARIANT, 5>), dim3(1), dim3(threads), 0, st, a); break;
    case 10:
      hipLaunchKernelGGL((k_solve_rr<VARIANT, 10>), dim3(1), dim3(threads), 0, st, a);
      break;
    case 20:
      hipLaunchKernelGGL((k_solve_rr<VARIANT, 20>), dim3(1), dim3(threads), 0, st, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_solve_rr_many(const Slot* slots, const int* idx, int n, hipStream_t st) {
  if (n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_solve_rr_many, dim3(n), dim3(kRrThreads), 0, st, slots, idx);
  return hipGetLastError();
}

hipError_t launch_solve_rr(int variant, const RrArgs& a, int threads, hipStream_t st) {
  const int rows = rr_rows(a.g.nx, a.g.ny);
  if (threads < kWave || threads > kRrThreads || threads % kWave || !rows ||
      rr_threads(a.g.nx, a.g.ny, rows) > threads || !a.b || !a.x || !a.out)
    return hipErrorInvalidValue;
  return variant == 1 ? launch_v<1>(a, rows, threads, st) : launch_v<0>(a, rows, threads, st);
}

}  // namespace cgk
