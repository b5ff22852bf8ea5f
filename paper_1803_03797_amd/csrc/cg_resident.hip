// cg_resident.hip - the iteration loop of a mid-size solve in one launch, its
// vectors held in registers across many compute units.
//
// A solve whose vectors fit the chip's registers spends its time elsewhere
// when every pass is a launch: at 300 x 190 the vectors are 0.5 MB and a
// classic iteration takes two launches of 4.7 us each, at 1024^2 a pipelined
// iteration streams 88 MB through the memory-side cache in 18 us.  Here one
// launch runs up to `budget` iterations.  Every wavefront keeps H strips (of
// R rows x 64 CPL columns) of each vector in registers from the first
// iteration to the last; what crosses work-groups is the boundary rows and
// columns and one partial sum per tile and dot product.  Solves to 1e-8, us per
// iteration, by passes / resident: 129 x 128 classic 9.7 / 2.95, pipelined 6.2 /
// 2.26; 300 x 190 9.6 / 3.3 and 6.3 / 2.85; 512^2 9.8 / 4.5 and 7.7 / 3.95;
// 1024^2 17.3 / 7.4 and 18.2 / 6.8; the FP32 inner iteration at 2048^2 25.6 /
// 9.8.  What is left is the meetings (one of 256 work-groups over the XCDs
// takes 5500 of a classic half-iteration's 8800 cycles at 1024^2) and the
// dependent chain around them.
//
// Exchange.  Work-groups meet once per reduction, without atomics that modify
// memory and without fences: everything exchanged is written as 64-bit words
// that hold 32 bits of data and the 32-bit number of the meeting, by relaxed
// agent-scope stores, and read by relaxed agent-scope loads until the number
// is right.  A word is its own flag, so no order between stores is assumed.
// (Agent-scope release / acquire fences would write back and invalidate the
// L2 on gfx950.)  Two buffers alternate: a work-group writes meeting n + 2
// only after it has seen every work-group's meeting n + 1, which each of them
// writes after reading all of meeting n.
//
// Near and far.  Where the work-groups of a solve fit one XCD they are placed
// there (every eighth work-group of the launch) and store their words at
// work-group scope: the words then stop at the L2 they share, where the polls
// (agent scope, past the L1) find them.  A meeting of 64 work-groups, and
// nothing else, takes 1100 cycles so, 3900 with agent-scope stores, and 2600
// to 4500 for 72 to 256 work-groups spread over the XCDs.  The placement is
// checked (the work-groups exchange their XCD numbers first, at agent scope);
// where it does not hold the solve is abandoned before its first meeting.
//
// Every wait is bounded: all work-groups of a solve must be on the device
// together, which the host ensures by the size of the launch, but another
// process, or another stream's long kernel, may hold the compute units.  A
// work-group that sees no progress for `spin` polls marks the solve as abandoned
// and ends; the others, waiting in the same meeting, then do the same, and the
// host runs the solve by passes.  (Looking at the mark while polling took 2 % of
// an iteration and ended a wait no sooner.)
//
// Results are those of the passes, bit for bit: the same tiles, lane order,
// butterflies, tile order and scalar recurrences.  x is updated every
// iteration, the same two fmas in the same order as the deferred update of
// the passes.
#include "cg_device.h"
#include "cg_internal.h"

namespace cgk {

namespace {

constexpr int kResWaves = kWavesPerTile;

// The exchange area is addressed as global memory: through a pointer read from
// memory the compiler would use flat accesses, which also occupy the LDS
// counter.
typedef __attribute__((address_space(1))) char* GlobalBytes;
typedef __attribute__((address_space(1))) uint64_t* GlobalWords;

// Words at a uniform base and a 32-bit byte offset (one register a word and
// no 64-bit address arithmetic), `k` words on.  NEAR: all readers share this
// XCD's L2.
template <bool NEAR>
__device__ __forceinline__ void put(GlobalBytes base, uint32_t off, int k, uint32_t tag,
                                    uint32_t bits) {
  const uint64_t v = (uint64_t)tag << 32 | bits;
  const GlobalWords w = (GlobalWords)(base + off) + k;
  if constexpr (NEAR) __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t get(GlobalBytes base, uint32_t off, int k) {
  // the sum base + offset is formed by the load itself, not kept across polls
  asm volatile("" : "+v"(off));
  return __hip_atomic_load((GlobalWords)(base + off) + k, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// A structure every lane reads alike, in scalar registers.
template <typename S>
__device__ __forceinline__ S load_uniform(const S* p) {
  static_assert(sizeof(S) % 16 == 0, "loaded as uint4");
  constexpr int N = sizeof(S) / 4;
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
  S s;
  __builtin_memcpy(&s, u, sizeof(S));
  return s;
}

// Words of one value: 32 bits each.
template <typename T>
constexpr int kWords = (int)sizeof(T) / 4;

__device__ __forceinline__ uint32_t word_of(double v, int k) {
  return (uint32_t)(k ? __double2hiint(v) : __double2loint(v));
}
__device__ __forceinline__ uint32_t word_of(float v, int) { return __float_as_uint(v); }

// The exchange area of one solve, after a header of one line (its first word:
// abandoned).  XCD numbers: a word per work-group.  Partials: [buffer]
// [work-group], word (tile of the work-group * D + slot) * 2 + half, packed
// near and one 128-byte line to a work-group far (a line with one writer: a
// meeting of 72 work-groups with sixteen 8-byte writers to a line took 3975
// cycles against 2618, of 256 6353 against 4476); rows: [buffer][work-group]
// [top, bottom][column, half][lane]; columns: [buffer][work-group][west, east]
// [half][row].
constexpr int kLine = 16;  // words

template <typename T, int CPL, int NR>
struct Area {
  static constexpr int kRow = kWords<T> * CPL * kWave;      // one boundary row
  static constexpr int kCol = kWords<T> * kResWaves * NR;   // one boundary column
  GlobalBytes xcd;                 // then the partials, the rows and the columns
  uint32_t xcd_b, part_b, rows_b, cols_b;  // bytes of one buffer
  uint32_t line;                   // bytes between two work-groups' partials
  __device__ __forceinline__ Area(uint64_t* sync, uint32_t n, uint32_t line_words) {
    xcd = (GlobalBytes)(sync + kLine);
    xcd_b = (n + kLine - 1) / kLine * kLine * 8;
    part_b = n * kLine * 8;
    rows_b = n * 2 * kRow * 8;
    cols_b = n * 2 * kCol * 8;
    line = line_words * 8;
  }
};

template <typename T, int CPL, int NR>
struct ResLds {
  Row<T, CPL> halo[kResWaves][2][kWave];  // every wavefront's first and last row
  T col[kResWaves][kWave];                // edge columns: side * 32 + row
  double strip[kResWaves * NR * 2];       // strip sums (at most NR strips a wavefront)
  double cross[kResWaves * 2];
  int dead;
};

// A wavefront's place in the grid.
struct Place {
  int lane, wave, bx, by, nby, wg;
  int c, ct;     // first column of the lane, of the tile
  int j0, rows;  // first row of the wavefront, rows of it inside the grid
  int valid;     // columns of the lane inside the grid (may be <= 0)
  bool whole;    // all of the wavefront's cells are inside the grid
  int side, row; // column exchange: lanes 0.. the west column's rows, 32.. the east's
};

template <int CPL, int R, int H>
__device__ __forceinline__ Place place_of(const Geo& g, int wg, int nby) {
  constexpr int NR = R * H;
  static_assert(NR <= 32, "the rows of a wavefront share its two half-waves");
  Place p;
  p.lane = threadIdx.x & (kWave - 1);
  p.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  p.wg = wg;
  p.bx = wg % g.ntx;
  p.by = wg / g.ntx;
  p.nby = nby;
  p.ct = p.bx * (kWave * CPL);
  p.c = p.ct + p.lane * CPL;
  p.j0 = (p.by * kResWaves + p.wave) * NR;
  p.rows = min(max(g.ny - p.j0, 0), NR);
  p.valid = g.nx - p.c;
  p.whole = p.rows == NR && p.ct + kWave * CPL <= g.nx;
  p.side = p.lane >> 5;
  p.row = p.lane & 31;
  return p;
}

// What a wavefront needs of its surroundings to apply the stencil: the rows
// above and below it and, of every row, the value left of lane 0 (in lanes
// 0-31) and right of lane 63 (in lanes 32-63).
template <typename T, int CPL, int NR>
struct Around {
  Row<T, CPL> top, bot;
  T col[NR];
};

template <typename T, int CPL, int NR>
__device__ __forceinline__ void load_rows(const T* V, const Geo& g, const Place& p,
                                          Row<T, CPL> (&v)[NR]) {
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    v[i] = zrow<T, CPL>();
    if (i < p.rows) v[i] = ldrow<T, CPL>(V + (size_t)(p.j0 + i) * g.pitch + p.c);
  }
}

template <typename T, int CPL, int NR>
__device__ __forceinline__ void store_rows(T* V, const Geo& g, const Place& p,
                                           const Row<T, CPL> (&v)[NR]) {
#pragma unroll
  for (int i = 0; i < NR; ++i)
    if (i < p.rows) strow<T, CPL>(V + (size_t)(p.j0 + i) * g.pitch + p.c, v[i], p.valid);
}

// The surroundings as they are in memory before the launch.
template <typename T, int CPL, int NR>
__device__ __forceinline__ Around<T, CPL, NR> load_around(const T* V, const Geo& g, const Place& p) {
  Around<T, CPL, NR> h;
  h.top = zrow<T, CPL>();
  h.bot = zrow<T, CPL>();
  if (p.j0 > 0 && p.j0 - 1 < g.ny)
    h.top = ldrow<T, CPL>(V + (size_t)(p.j0 - 1) * g.pitch + p.c);
  if (p.j0 + NR < g.ny) h.bot = ldrow<T, CPL>(V + (size_t)(p.j0 + NR) * g.pitch + p.c);
  const int col = p.side ? p.ct + kWave * CPL : p.ct - 1;
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    h.col[i] = T(0);
    if (i < p.rows && (p.side ? p.bx + 1 < g.ntx : p.bx > 0))
      h.col[i] = V[(size_t)(p.j0 + i) * g.pitch + col];
  }
  return h;
}

// What a thread reads and writes at every meeting: byte offsets within one
// buffer of the area's parts.
template <int NP>
struct Post {
  uint32_t poll[NP];        // partials of tiles tid + 256 e (first of two words)
  uint32_t put_row, put_col, get_row, get_col;
  int ne;                   // tiles this thread polls (of the first NP)
  bool has_row, has_col;    // a neighbouring work-group is above / below, beside
};

template <int H, int D>
__device__ __forceinline__ uint32_t partial_at(const Geo& g, uint32_t line, int t) {
  const int ty = t / g.ntx, bx = t % g.ntx;
  return (uint32_t)((ty / H) * g.ntx + bx) * line + (uint32_t)((ty % H) * D * 2) * 8;
}

template <typename T, int CPL, int R, int H, int D, int NP>
__device__ __forceinline__ Post<NP> post_of(const Geo& g, const Place& p, uint32_t line) {
  constexpr int NR = R * H;
  using A = Area<T, CPL, NR>;
  static_assert(H * D * 2 <= kLine, "the partials of a work-group fill one line");
  Post<NP> o;
  o.ne = 0;
#pragma unroll
  for (int e = 0; e < NP; ++e) {
    const int t = (int)threadIdx.x + e * kGroup;
    o.poll[e] = 0;
    if (t < g.tiles) {
      o.poll[e] = partial_at<H, D>(g, line, t);
      o.ne = e + 1;
    }
  }
  const bool up = p.wave == 0 && p.by > 0;
  const bool down = p.wave == kResWaves - 1 && p.by + 1 < p.nby;
  o.has_row = up || down;
  o.put_row = (uint32_t)((p.wg * 2 + (down ? 1 : 0)) * A::kRow + p.lane) * 8;
  o.get_row = 0;
  if (up) o.get_row = (uint32_t)(((p.wg - g.ntx) * 2 + 1) * A::kRow + p.lane) * 8;
  if (down) o.get_row = (uint32_t)(((p.wg + g.ntx) * 2) * A::kRow + p.lane) * 8;
  o.has_col = p.row < NR && (p.side ? p.bx + 1 < g.ntx : p.bx > 0);
  o.put_col = (uint32_t)((p.wg * 2 + p.side) * A::kCol + p.wave * NR + p.row) * 8;
  o.get_col = 0;
  if (o.has_col)
    o.get_col = (uint32_t)(((p.side ? p.wg + 1 : p.wg - 1) * 2 + (1 - p.side)) * A::kCol +
                           p.wave * NR + p.row) * 8;
  return o;
}

__device__ __forceinline__ uint32_t off_tag(uint64_t w, uint32_t tag) {
  return (uint32_t)(w >> 32) ^ tag;
}

__device__ __forceinline__ double join(uint64_t lo, uint64_t hi) {
  return __hiloint2double((int)hi, (int)lo);
}

// One meeting.  lv: the lane's sums of its H strips and D dot products.  With
// HALO, v are the wavefront's rows of the vector whose boundary is exchanged
// and `h` receives its new surroundings.  sum: the cross-tile sums; mine: the
// partial published by the thread (threads below 2 H D: tile and slot
// tid / 2).  False: abandoned.
template <typename T, int CPL, int R, int H, int D, bool HALO, bool NEAR, int NP>
__device__ __forceinline__ bool meet(const Area<T, CPL, R * H>& m, const Post<NP>& o,
                                     const Place& p,
                                     ResLds<T, CPL, R * H>& L, const Geo& g, int spin,
                                     uint32_t tag, const double (&lv)[H][D],
                                     const Row<T, CPL> (&v)[R * H], Around<T, CPL, R * H>& h,
                                     double (&sum)[2], double& mine) {
  constexpr int NR = R * H, NW = kWords<T>;
  const int tid = threadIdx.x;
  const uint32_t buf = __builtin_amdgcn_readfirstlane(tag & 1);
  // opaque scalar bases: else the compiler adds each thread's offset to the
  // part both buffers share and keeps a 64-bit address per word in registers
  GlobalBytes part = m.xcd + m.xcd_b + buf * m.part_b;
  GlobalBytes rows = m.xcd + m.xcd_b + 2 * m.part_b + buf * m.rows_b;
  GlobalBytes cols = m.xcd + m.xcd_b + 2 * m.part_b + 2 * m.rows_b + buf * m.cols_b;
  asm("" : "+s"(part), "+s"(rows), "+s"(cols));
  const bool last = p.wave != 0;  // a wavefront with a row to exchange: the bottom one
  if constexpr (HALO) {
    // the boundary first: it travels while the sums are formed
    L.halo[p.wave][0][p.lane] = v[0];
    L.halo[p.wave][1][p.lane] = v[NR - 1];
    if (o.has_row) {
#pragma unroll
      for (int k = 0; k < CPL; ++k)
#pragma unroll
        for (int w = 0; w < NW; ++w)
          put<NEAR>(rows, o.put_row, (k * NW + w) * kWave, tag,
              word_of(last ? v[NR - 1].e[k] : v[0].e[k], w));
    }
    if (p.lane == 0 || p.lane == kWave - 1) {
#pragma unroll
      for (int i = 0; i < NR; ++i)
        L.col[p.wave][p.side * 32 + i] = p.side ? v[i].e[CPL - 1] : v[i].e[0];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    if (o.has_col) {
      const T c = L.col[p.wave][p.lane];
#pragma unroll
      for (int w = 0; w < NW; ++w) put<NEAR>(cols, o.put_col, w * kResWaves * NR, tag, word_of(c, w));
    }
  }
  double sv[H][D];
#pragma unroll
  for (int s = 0; s < H; ++s)
#pragma unroll
    for (int d = 0; d < D; ++d) sv[s][d] = wave_sum_valu(lv[s][d]);
  if (p.lane == 0) {
#pragma unroll
    for (int s = 0; s < H; ++s)
#pragma unroll
      for (int d = 0; d < D; ++d) L.strip[(p.wave * H + s) * D + d] = sv[s][d];
  }
  lds_barrier();
  // the H tiles' partials: their four strips in order, one word a thread
  if (tid < 2 * H * D) {
    const int hh = (tid >> 1) / D, d = (tid >> 1) % D;
    double t = L.strip[(hh * kWavesPerTile) * D + d];
#pragma unroll
    for (int w = 1; w < kWavesPerTile; ++w) t = t + L.strip[(hh * kWavesPerTile + w) * D + d];
    mine = t;
    put<NEAR>(part, (uint32_t)p.wg * m.line + tid * 8, 0, tag, word_of(t, tid & 1));
  }
  bool alive = true;
  const uint64_t want = (uint64_t)tag << 32;
  if constexpr (HALO) {
    if (p.wave > 0) h.top = L.halo[p.wave - 1][1][p.lane];
    if (p.wave + 1 < kResWaves) h.bot = L.halo[p.wave + 1][0][p.lane];
  }
  // poll: the partials of all tiles and what this wavefront takes of the
  // neighbouring work-groups, all loads of a round in flight together
  double acc[D];
#pragma unroll
  for (int d = 0; d < D; ++d) acc[d] = 0.0;
  T col = T(0);  // lane l: side l / 32, row l % 32
  for (;;) {
    uint64_t lo[NP][D], hi[NP][D];
    uint32_t bad = 0;
#pragma unroll
    for (int e = 0; e < NP; ++e)
#pragma unroll
      for (int d = 0; d < D; ++d) {
        lo[e][d] = hi[e][d] = want;
        if (e < o.ne) {
          lo[e][d] = get(part, o.poll[e], d * 2);
          hi[e][d] = get(part, o.poll[e], d * 2 + 1);
        }
      }
    if constexpr (HALO) {
      uint64_t cw[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) cw[w] = want;
      if (o.has_col) {
#pragma unroll
        for (int w = 0; w < NW; ++w) cw[w] = get(cols, o.get_col, w * kResWaves * NR);
      }
      if (o.has_row) {
        uint64_t rw[CPL * NW];
        Row<T, CPL> rr;
#pragma unroll
        for (int w = 0; w < CPL * NW; ++w) rw[w] = get(rows, o.get_row, w * kWave);
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
          if constexpr (NW == 2) rr.e[k] = join(rw[2 * k], rw[2 * k + 1]);
          else rr.e[k] = __uint_as_float((unsigned)rw[k]);
        }
#pragma unroll
        for (int w = 0; w < CPL * NW; ++w) bad |= off_tag(rw[w], tag);
        if (last) h.bot = rr;
        else h.top = rr;
      }
#pragma unroll
      for (int w = 0; w < NW; ++w) bad |= off_tag(cw[w], tag);
      if constexpr (NW == 2) col = join(cw[0], cw[1]);
      else col = __uint_as_float((unsigned)cw[0]);
    }
#pragma unroll
    for (int e = 0; e < NP; ++e)
#pragma unroll
      for (int d = 0; d < D; ++d) bad |= off_tag(lo[e][d], tag) | off_tag(hi[e][d], tag);
    if (bad == 0) {
#pragma unroll
      for (int e = 0; e < NP; ++e)
#pragma unroll
        for (int d = 0; d < D; ++d)
          if (e < o.ne) acc[d] = acc[d] + join(lo[e][d], hi[e][d]);
      break;
    }
    if (--spin < 0) {
      alive = false;
      break;
    }
  }
  // grids of more tiles: the rest, one after the other
  for (int k = tid + NP * kGroup; k < g.tiles && alive; k += kGroup) {
    const uint32_t q = partial_at<H, D>(g, m.line, k);
    uint64_t lo[D], hi[D];
    uint32_t bad;
    do {
      bad = 0;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        lo[d] = get(part, q, d * 2);
        hi[d] = get(part, q, d * 2 + 1);
        bad |= off_tag(lo[d], tag) | off_tag(hi[d], tag);
      }
      if (--spin < 0) alive = false;
    } while (bad != 0 && alive);
#pragma unroll
    for (int d = 0; d < D; ++d) acc[d] = acc[d] + join(lo[d], hi[d]);
  }
  if (!alive) L.dead = 1;
  if constexpr (HALO) L.col[p.wave][p.lane] = col;
#pragma unroll
  for (int d = 0; d < D; ++d) acc[d] = wave_sum_valu(acc[d]);
  if (p.lane == 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) L.cross[p.wave * D + d] = acc[d];
  }
  lds_barrier();
  if constexpr (HALO) {
#pragma unroll
    for (int i = 0; i < NR; ++i) h.col[i] = L.col[p.wave][p.side * 32 + i];
  }
#pragma unroll
  for (int d = 0; d < D; ++d) {
    double t = L.cross[d];
#pragma unroll
    for (int w = 1; w < kWavesPerTile; ++w) t = t + L.cross[w * D + d];
    sum[d] = uniform(t);
  }
  return __builtin_amdgcn_readfirstlane(L.dead) == 0;
}

// Whether the solve's work-groups share an XCD; tag: not used by any meeting.
template <typename T, int CPL, int NR>
__device__ __forceinline__ bool share_xcd(const Area<T, CPL, NR>& m, const Place& p, int n,
                                          int spin, uint32_t tag, int* dead) {
  const uint32_t mine =
      __builtin_amdgcn_s_getreg(20 | (31 << 11));  // hardware register XCC_ID, 32 bits
  const uint64_t want = (uint64_t)tag << 32 | mine;
  if (threadIdx.x == 0) put<false>(m.xcd, (uint32_t)p.wg * 8, 0, tag, mine);
  bool same = true;
  for (int k = threadIdx.x; k < n && same; k += kGroup) {
    uint64_t v;
    do {
      v = get(m.xcd, (uint32_t)k * 8, 0);
      if (--spin < 0) same = false;
    } while ((v >> 32) != tag && same);
    same = same && v == want;
  }
  if (!same) *dead = 1;
  lds_barrier();
  return __builtin_amdgcn_readfirstlane(*dead) == 0;
}

__device__ __forceinline__ void give_up(uint64_t* sync) {
  if (threadIdx.x == 0)
    __hip_atomic_store(sync, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The descriptor read again where a launch ends: its fields (and the state's
// that no recurrence changes) would otherwise hold scalar registers, and
// spill, through the whole loop.
__device__ __forceinline__ ResSolve again(const ResSolve* a) {
  asm volatile("" : "+s"(a));
  return load_uniform(a);
}

// Likewise the wavefront's place, or the addresses of its rows would be kept
// from the entry to the exit.
template <int CPL, int R, int H>
__device__ __forceinline__ Place place_again(const Geo& g, int wg) {
  asm volatile("" : "+s"(wg));
  return place_of<CPL, R, H>(g, wg, (g.nty + H - 1) / H);
}

__device__ __forceinline__ void write_state(const ResSolve& a, const State& s, int kind) {
  State o = *a.st_in;
  o.gamma = s.gamma;
  o.gamma0 = s.gamma0;
  o.delta = s.delta;
  o.alpha = s.alpha;
  o.beta = s.beta;
  o.bb = s.bb;
  o.thr = s.thr;
  o.thr_in = s.thr_in;
  o.k = s.k;
  o.kin = s.kin;
  o.status = s.status;
  o.flags = s.flags;
  o.kind = kind;
  *a.st_out = o;
}

template <typename T, int CPL>
__device__ __forceinline__ Row<T, CPL> minus_zero() {
  Row<T, CPL> v;
#pragma unroll
  for (int k = 0; k < CPL; ++k) v.e[k] = T(-0.0);
  return v;
}

// The scalars of an iteration.  The loop forms them itself, with the
// operations of transition<>, as long as nothing ends the solve; everything
// else (the first iteration, a stop, a breakdown) goes through transition<>.
struct Scalars {
  double gamma, alpha, beta, thr;
  int k, maxit;
  __device__ __forceinline__ void to(State& s, int kin0, int k0) const {
    s.gamma = gamma;
    s.delta = gamma;
    s.alpha = alpha;
    s.beta = beta;
    s.k = k;
    s.kin = kin0 + (k - k0);
  }
  // stop_code(g, ...) == ST_RUNNING
  __device__ __forceinline__ bool goes_on(double g) const {
    return g > thr && g < __builtin_huge_val() && k < maxit;
  }
};

// Row i of A v.
template <typename T, int CPL>
__device__ __forceinline__ Row<T, CPL> stencil_row(const Row<T, CPL>& S, const Row<T, CPL>& C,
                                                   const Row<T, CPL>& N, T e) {
  Row<T, CPL> W, E, o;
  west_east<T, CPL>(C, e, e, W, E);
#pragma unroll
  for (int k = 0; k < CPL; ++k) o.e[k] = st5(C.e[k], W.e[k], E.e[k], S.e[k], N.e[k]);
  return o;
}

// Cells outside the grid are held at zero through every iteration: A v is
// cleared there, in the wavefronts that have any (p.whole: none).
template <typename T, int CPL>
__device__ __forceinline__ void clip(Row<T, CPL>& v, const Place& p, int i) {
#pragma unroll
  for (int k = 0; k < CPL; ++k) v.e[k] = (i < p.rows && k < p.valid) ? v.e[k] : T(0);
}

// The lane's sums over the rows of strip s in the order of the passes: down
// the strip, or up it for the odd strips of a tile (ALT, the classic passes).
// With an odd H the direction depends on the wavefront; the empty asm keeps the
// two directions apart (merged, they index the rows at run time, which puts them
// in scratch memory).
template <int R, int H, bool ALT, class F>
__device__ __forceinline__ void strip_rows(const Place& p, int s, F f) {
  const bool up = ALT && (((p.wave * H + s) & 1) != 0);
  if (up) {
#pragma unroll
    for (int i = R - 1; i >= 0; --i) f(s * R + i);
    if (H & 1) asm volatile("; up");
  } else {
#pragma unroll
    for (int i = 0; i < R; ++i) f(s * R + i);
    if (H & 1) asm volatile("; down");
  }
}

// Classic CG (T double: K_CG1 / K_CG2; float: the refinement's K_CG1F /
// K_CG2F) from an even iteration.  Bound by the two meetings of an iteration.
template <typename T, int CPL, int R, int H, bool NEAR>
__device__ __forceinline__ void resident_cg(const ResSolve* pa, int wg, char* raw) {
  constexpr int NR = R * H;
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int K1 = F32 ? K_CG1F : K_CG1, K2 = F32 ? K_CG2F : K_CG2;
  using L_t = ResLds<T, CPL, NR>;
  L_t& L = *reinterpret_cast<L_t*>(raw);
  const ResSolve a = load_uniform(pa);
  const Geo g = a.g;
  const int nby = (g.nty + H - 1) / H;
  const Place p = place_of<CPL, R, H>(g, wg, nby);
  constexpr int NP = NEAR ? 1 : H;
  const Area<T, CPL, NR> m(a.sync, nby * g.ntx, NEAR ? 2 * H * 1 : kLine);
  const Post<NP> o = post_of<T, CPL, R, H, 1, NP>(g, p, m.line);
  Row<T, CPL> r[NR], d[NR], s[NR], x[NR];
  Around<T, CPL, NR> ra, pa_;
  auto vectors = [](const ResSolve& q, T*& rv, T*& xv, T*& pv) {
    if constexpr (F32) {
      rv = q.rf;
      xv = q.df;
      pv = q.pf;
    } else {
      rv = q.r;
      xv = q.x;
      pv = q.pc;
    }
  };
  {
    T *Rv, *Xv, *Pv;
    vectors(a, Rv, Xv, Pv);
    load_rows<T, CPL, NR>(Rv, g, p, r);
    load_rows<T, CPL, NR>(Pv, g, p, d);
    load_rows<T, CPL, NR>(Xv, g, p, x);
    ra = load_around<T, CPL, NR>(Rv, g, p);
    pa_ = load_around<T, CPL, NR>(Pv, g, p);
  }
  State st = load_state_uniform(a.st_in);
  if (threadIdx.x == 0) L.dead = 0;
  double sum[2] = {0.0, 0.0};
  if (!F32 && (st.flags & F_BB_PENDING)) cross_tile_sum<2>(a.part_in, g.tiles, sum, L.cross);
  else cross_tile_sum<1>(a.part_in, g.tiles, sum, L.cross);
  sum[0] = uniform(sum[0]);
  sum[1] = uniform(sum[1]);
  const uint32_t seq = a.seq;
  const int spin = a.spin, budget = a.budget;
  if constexpr (NEAR)
    if (!share_xcd(m, p, nby * g.ntx, spin, seq, &L.dead)) return give_up(again(pa).sync);
  uint32_t tag = seq;
  double mine = 0.0;
  Sc sc;
  bool stopped = !uniform_flag(transition<K1>(st, sum, sc));
  Scalars c{st.gamma, st.alpha, st.beta, F32 ? st.thr_in : st.thr, st.k, st.maxit};
  const int k0 = c.k, kin0 = st.kin;
  if (uniform_flag(sc.first != 0)) {
    // p = r: beta is 0, and 0 * -0 + r is r bit for bit
#pragma unroll
    for (int i = 0; i < NR; ++i) d[i] = minus_zero<T, CPL>();
    pa_.top = pa_.bot = minus_zero<T, CPL>();
#pragma unroll
    for (int i = 0; i < NR; ++i) pa_.col[i] = T(-0.0);
  }
  for (int it = 0; !stopped;) {
    // p = r + beta p, here and around; s = A p; (p, s)
    const T be = T(c.beta);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      pa_.col[i] = fma(be, pa_.col[i], ra.col[i]);
#pragma unroll
      for (int k = 0; k < CPL; ++k) d[i].e[k] = fma(be, d[i].e[k], r[i].e[k]);
    }
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      pa_.top.e[k] = fma(be, pa_.top.e[k], ra.top.e[k]);
      pa_.bot.e[k] = fma(be, pa_.bot.e[k], ra.bot.e[k]);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i)
      s[i] = stencil_row<T, CPL>(i ? d[i ? i - 1 : 0] : pa_.top, d[i],
                                 i + 1 < NR ? d[i + 1 < NR ? i + 1 : i] : pa_.bot, pa_.col[i]);
    if (!p.whole) {
#pragma unroll
      for (int i = 0; i < NR; ++i) clip<T, CPL>(s[i], p, i);
    }
    double lv[H][1];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      double a0[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) a0[k] = 0.0;
      strip_rows<R, H, true>(p, h, [&](int i) {
#pragma unroll
        for (int k = 0; k < CPL; ++k) a0[k] = fma((double)d[i].e[k], (double)s[i].e[k], a0[k]);
      });
      lv[h][0] = fold<CPL>(a0);
    }
    if (!meet<T, CPL, R, H, 1, false, NEAR>(m, o, p, L, g, spin, ++tag, lv, r, ra, sum, mine))
      return give_up(again(pa).sync);
    if (!(sum[0] > 0.0 && sum[0] < __builtin_huge_val())) {
      c.to(st, kin0, k0);
      (void)transition<K2>(st, sum, sc);  // a breakdown
      stopped = true;
      break;
    }
    // x += alpha p; r -= alpha s; (r, r)
    c.alpha = c.gamma / sum[0];
    c.k += 1;
    const T al = T(c.alpha), nal = -al;
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int k = 0; k < CPL; ++k) r[i].e[k] = fma(nal, s[i].e[k], r[i].e[k]);
#pragma unroll
    for (int h = 0; h < H; ++h) {
      double a0[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) a0[k] = 0.0;
      strip_rows<R, H, true>(p, h, [&](int i) {
#pragma unroll
        for (int k = 0; k < CPL; ++k) a0[k] = fma((double)r[i].e[k], (double)r[i].e[k], a0[k]);
      });
      lv[h][0] = fold<CPL>(a0);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i)
#pragma unroll
      for (int k = 0; k < CPL; ++k) x[i].e[k] = fma(al, d[i].e[k], x[i].e[k]);
    if (!meet<T, CPL, R, H, 1, true, NEAR>(m, o, p, L, g, spin, ++tag, lv, r, ra, sum, mine))
      return give_up(again(pa).sync);
    ++it;
    if (it >= budget && !((F32 ? kin0 + (c.k - k0) : c.k) & 1)) {
      c.to(st, kin0, k0);
      break;
    }
    if (!c.goes_on(sum[0])) {
      c.to(st, kin0, k0);
      if (!uniform_flag(transition<K1>(st, sum, sc))) {
        stopped = true;
        break;
      }
    }
    c.beta = sum[0] / c.gamma;
    c.gamma = sum[0];
  }
  // the outputs may be the inputs: a launch that stops before any meeting
  // holds one first, after which every work-group has read its inputs
  if (tag == seq) {
    const double none[H][1] = {};
    double mine0;
    if (!meet<T, CPL, R, H, 1, false, NEAR>(m, o, p, L, g, spin, ++tag, none, r, ra, sum, mine0))
      return give_up(again(pa).sync);
  }
  const ResSolve z = again(pa);
  const Geo gz = z.g;
  const Place pz = place_again<CPL, R, H>(gz, wg);
  T *Rv, *Xv, *Pv;
  vectors(z, Rv, Xv, Pv);
  store_rows<T, CPL, NR>(Xv, gz, pz, x);
  if (!stopped) {
    store_rows<T, CPL, NR>(Rv, gz, pz, r);
    store_rows<T, CPL, NR>(Pv, gz, pz, d);
    const int ty = pz.by * H + (int)(threadIdx.x >> 1);
    if (threadIdx.x < 2 * H && !(threadIdx.x & 1) && ty < gz.nty)
      z.part_out[ty * gz.ntx + pz.bx] = mine;
  }
  if (wg == 0 && threadIdx.x == 0)
    write_state(z, st, !stopped ? K1 : F32 ? K_REF_UPDATE
                                 : st.status == ST_ZERO_RHS ? K_DONE : K_RESID);
}

// Pipelined CG (K_PCG / K_PCGX) from an even iteration: one meeting an
// iteration.
template <int R, int H, bool NEAR>
__device__ __forceinline__ void resident_pcg(const ResSolve* pa, int wg, char* raw) {
  constexpr int NR = R * H, CPL = 2;
  using T = double;
  using L_t = ResLds<T, CPL, NR>;
  L_t& L = *reinterpret_cast<L_t*>(raw);
  const ResSolve a = load_uniform(pa);
  const Geo g = a.g;
  const int nby = (g.nty + H - 1) / H;
  const Place p = place_of<CPL, R, H>(g, wg, nby);
  constexpr int NP = NEAR ? 1 : H;
  const Area<T, CPL, NR> m(a.sync, nby * g.ntx, NEAR ? 2 * H * 2 : kLine);
  const Post<NP> o = post_of<T, CPL, R, H, 2, NP>(g, p, m.line);
  Row<T, CPL> r[NR], w[NR], z[NR], q[NR], d[NR], x[NR];
  load_rows<T, CPL, NR>(a.r, g, p, r);
  load_rows<T, CPL, NR>(a.w, g, p, w);
  load_rows<T, CPL, NR>(a.z, g, p, z);
  load_rows<T, CPL, NR>(a.q, g, p, q);
  load_rows<T, CPL, NR>(a.p, g, p, d);
  load_rows<T, CPL, NR>(a.x, g, p, x);
  Around<T, CPL, NR> wa = load_around<T, CPL, NR>(a.w, g, p);
  State st = load_state_uniform(a.st_in);
  if (threadIdx.x == 0) L.dead = 0;
  double sum[2];
  cross_tile_sum<2>(a.part_in, g.tiles, sum, L.cross);
  sum[0] = uniform(sum[0]);
  sum[1] = uniform(sum[1]);
  const uint32_t seq = a.seq;
  const int spin = a.spin, budget = a.budget;
  if constexpr (NEAR)
    if (!share_xcd(m, p, nby * g.ntx, spin, seq, &L.dead)) return give_up(again(pa).sync);
  uint32_t tag = seq;
  double mine = 0.0;
  Sc sc;
  bool stopped = !uniform_flag(transition<K_PCG>(st, sum, sc));
  Scalars c{st.gamma, st.alpha, st.beta, st.thr, st.k, st.maxit};
  const int k0 = c.k;
  if (uniform_flag(sc.first != 0)) {
    // z = A w, q = w, p = r: beta is 0, and 0 * -0 + v is v bit for bit
#pragma unroll
    for (int i = 0; i < NR; ++i) z[i] = q[i] = d[i] = minus_zero<T, CPL>();
  }
  for (int it = 0; !stopped;) {
    const double al = c.alpha, nal = -al, be = c.beta;
    Row<T, CPL> S = wa.top;
    double lv[H][2];
#pragma unroll
    for (int h = 0; h < H; ++h) {
      double a0[CPL], a1[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) a0[k] = a1[k] = 0.0;
#pragma unroll
      for (int ii = 0; ii < R; ++ii) {
        const int i = h * R + ii;
        const Row<T, CPL> C = w[i];
        Row<T, CPL> nv = stencil_row<T, CPL>(
            S, C, i + 1 < NR ? w[i + 1 < NR ? i + 1 : i] : wa.bot, wa.col[i]);
        if (!p.whole) clip<T, CPL>(nv, p, i);
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
          z[i].e[k] = fma(be, z[i].e[k], nv.e[k]);
          q[i].e[k] = fma(be, q[i].e[k], C.e[k]);
          d[i].e[k] = fma(be, d[i].e[k], r[i].e[k]);
          r[i].e[k] = fma(nal, q[i].e[k], r[i].e[k]);
          w[i].e[k] = fma(nal, z[i].e[k], C.e[k]);
          a0[k] = fma(r[i].e[k], r[i].e[k], a0[k]);
          a1[k] = fma(w[i].e[k], r[i].e[k], a1[k]);
          x[i].e[k] = fma(al, d[i].e[k], x[i].e[k]);
        }
        S = C;
      }
      lv[h][0] = fold<CPL>(a0);
      lv[h][1] = fold<CPL>(a1);
    }
    if (!meet<T, CPL, R, H, 2, true, NEAR>(m, o, p, L, g, spin, ++tag, lv, w, wa, sum, mine))
      return give_up(again(pa).sync);
    ++it;
    if (it >= budget && !(c.k & 1)) {
      c.to(st, 0, k0);
      break;
    }
    const double be1 = sum[0] / c.gamma;
    const double den = sum[1] / sum[0] - be1 / c.alpha;
    if (c.goes_on(sum[0]) && den > 0.0 && den < __builtin_huge_val()) {
      c.beta = be1;
      c.alpha = 1.0 / den;
      c.gamma = sum[0];
      c.k += 1;
    } else {
      c.to(st, 0, k0);
      if (!uniform_flag(transition<K_PCG>(st, sum, sc))) {
        stopped = true;
        break;
      }
      c.beta = st.beta;
      c.alpha = st.alpha;
      c.gamma = st.gamma;
      c.k = st.k;
    }
  }
  if (tag == seq) {
    const double none[H][2] = {};
    double mine0;
    if (!meet<T, CPL, R, H, 2, false, NEAR>(m, o, p, L, g, spin, ++tag, none, r, wa, sum, mine0))
      return give_up(again(pa).sync);
  }
  const ResSolve y = again(pa);
  const Geo gy = y.g;
  const Place py = place_again<CPL, R, H>(gy, wg);
  store_rows<T, CPL, NR>(y.x, gy, py, x);
  if (!stopped) {
    store_rows<T, CPL, NR>(y.r, gy, py, r);
    store_rows<T, CPL, NR>(y.w, gy, py, w);
    store_rows<T, CPL, NR>(y.z, gy, py, z);
    store_rows<T, CPL, NR>(y.q, gy, py, q);
    store_rows<T, CPL, NR>(y.p, gy, py, d);
    const int hh = (int)(threadIdx.x >> 1) / 2, dd = (threadIdx.x >> 1) % 2, ty = py.by * H + hh;
    if (threadIdx.x < 4 * H && !(threadIdx.x & 1) && ty < gy.nty)
      y.part_out[(size_t)dd * gy.tiles + ty * gy.ntx + py.bx] = mine;
  }
  if (wg == 0 && threadIdx.x == 0)
    write_state(y, st, !stopped ? K_PCG : st.status == ST_ZERO_RHS ? K_DONE : K_RESID);
}

template <int KIND, int R, int H, bool NEAR>
__device__ __forceinline__ void resident(const ResSolve* a, int wg, char* raw) {
  if constexpr (KIND == 0) resident_cg<double, 2, R, H, NEAR>(a, wg, raw);
  else if constexpr (KIND == 1) resident_pcg<R, H, NEAR>(a, wg, raw);
  else resident_cg<float, 4, R, H, NEAR>(a, wg, raw);
}

template <int KIND, int NR>
constexpr size_t lds_bytes() {
  return KIND == 2 ? sizeof(ResLds<float, 4, NR>) : sizeof(ResLds<double, 2, NR>);
}

// KIND: 0 classic FP64, 1 pipelined FP64, 2 the refinement's inner solve.
// One solve: work-group blockIdx.x, near every eighth block's (block b runs on
// XCD b % 8).
template <int KIND, int R, int H, bool NEAR>
__global__ __launch_bounds__(kGroup) void k_resident(ResSolve one) {
  __shared__ alignas(16) char raw[lds_bytes<KIND, R * H>()];
  int wg = blockIdx.x;
  if (NEAR) {
    if (wg & 7) return;
    wg >>= 3;
  }
  // `one` is the kernel's only argument: read where it lies
  resident<KIND, R, H, NEAR>((const ResSolve*)__builtin_amdgcn_kernarg_segment_ptr(), wg, raw);
}

// The forms of k_resident_many, each a function of its own (inlined side by
// side they would share one register allocation, and spill).
typedef __attribute__((address_space(3))) char* LdsBytes;

template <int KIND, int H, bool NEAR>
__device__ __attribute__((noinline)) void resident_call(const ResSolve* a, int wg,
                                                        LdsBytes lds) {
  const uint64_t p = (uint64_t)a;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  resident<KIND, 2, H, NEAR>((const ResSolve*)((uint64_t)hi << 32 | lo),
                             __builtin_amdgcn_readfirstlane(wg), (char*)lds);
}

// Several solves, one listed work-group a block; a negative solve leaves its
// block idle.  One kernel for all forms, so that any two work-groups fit a
// compute unit (at most 256 registers): what the host counts by.
__global__ __launch_bounds__(kGroup, 2) void k_resident_many(const ResSolve* many,
                                                             const ResWg* wgs) {
  __shared__ alignas(16) char raw[lds_bytes<0, 8>()];
  static_assert(lds_bytes<2, 8>() <= lds_bytes<0, 8>(), "one size for both types");
  const ResWg e = wgs[blockIdx.x];
  const int i = __builtin_amdgcn_readfirstlane(e.solve);
  const int wg = __builtin_amdgcn_readfirstlane(e.wg);
  if (i < 0) return;
  const ResSolve* a = many + i;
  switch (__builtin_amdgcn_readfirstlane(a->form)) {
    case resident_form(0, 1, true): return resident_call<0, 1, true>(a, wg, (LdsBytes)raw);
    case resident_form(0, 2, true): return resident_call<0, 2, true>(a, wg, (LdsBytes)raw);
    case resident_form(0, 4, true): return resident_call<0, 4, true>(a, wg, (LdsBytes)raw);
    case resident_form(1, 1, true): return resident_call<1, 1, true>(a, wg, (LdsBytes)raw);
    case resident_form(1, 2, true): return resident_call<1, 2, true>(a, wg, (LdsBytes)raw);
    case resident_form(2, 1, true): return resident_call<2, 1, true>(a, wg, (LdsBytes)raw);
    case resident_form(2, 2, true): return resident_call<2, 2, true>(a, wg, (LdsBytes)raw);
    case resident_form(2, 4, true): return resident_call<2, 4, true>(a, wg, (LdsBytes)raw);
    case resident_form(0, 4, false): return resident_call<0, 4, false>(a, wg, (LdsBytes)raw);
    case resident_form(1, 2, false): return resident_call<1, 2, false>(a, wg, (LdsBytes)raw);
    case resident_form(2, 4, false): return resident_call<2, 4, false>(a, wg, (LdsBytes)raw);
  }
}

// The state each solve was left in; pad_ set: it was abandoned.
__global__ void k_resident_states(const ResSolve* many, int n, State* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  State s = *many[i].st_out;
  s.pad_ = many[i].sync[0] != 0;
  out[i] = s;
}

// The compiled shapes of one solve.  Strips of 2 rows cover the grids of up to
// about 1.5 times 1024 tiles.  Taller ones, which larger grids have, are there
// for the binary32 inner solve (four vectors of half the bytes), with as many
// strips as its registers take: of 3 rows 6 (1024 to 1366 tiles on 256
// work-groups), of 4 rows 4 or, from 1025 tiles, 5 (19 registers spilled; up to
// 1280 tiles).  us per iteration by passes / resident: 1792^2 21.2 / 9.3 (3
// rows), 2047^2 26.2 / 10.4, 2048^2 24.2 / 8.7 (4 rows, 4 strips), 2049^2 26.4 /
// 11.3 (5 strips), 2200^2 27.8 / 11.6.  Larger grids (from 2241^2) would need more
// rows a wavefront than fit.
using Kernel = void (*)(ResSolve);

template <int KIND, bool NEAR>
Kernel kernel_h(int rows, int strips) {
  if (rows == 2 && strips == 1) return k_resident<KIND, 2, 1, NEAR>;
  if (rows == 2 && strips == 2) return k_resident<KIND, 2, 2, NEAR>;
  // the pipelined solve of four strips takes a compute unit: what then fits one
  // XCD fits it with two strips as well
  if constexpr (KIND != 1 || !NEAR)
    if (rows == 2 && strips == 4) return k_resident<KIND, 2, 4, NEAR>;
  if constexpr (KIND == 2 && !NEAR) {
    if (rows == 3 && strips == 6) return k_resident<KIND, 3, 6, NEAR>;
    if (rows == 4 && strips == 4) return k_resident<KIND, 4, 4, NEAR>;
    if (rows == 4 && strips == 5) return k_resident<KIND, 4, 5, NEAR>;
  }
  return nullptr;
}

Kernel kernel_of(int kind, int rows, int strips, bool near) {
  switch (kind) {
    case 0: return near ? kernel_h<0, true>(rows, strips) : kernel_h<0, false>(rows, strips);
    case 1: return near ? kernel_h<1, true>(rows, strips) : kernel_h<1, false>(rows, strips);
    case 2: return near ? kernel_h<2, true>(rows, strips) : kernel_h<2, false>(rows, strips);
  }
  return nullptr;
}

}  // namespace

int resident_blocks_per_cu(int kind, int rows, int strips, bool near) {
  const Kernel k = kernel_of(kind, rows, strips, near);
  int n = 0;
  if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, kGroup, 0) != hipSuccess)
    return 0;
  return n;
}

int resident_many_blocks_per_cu() {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_resident_many, kGroup, 0) != hipSuccess)
    return 0;
  return n;
}

bool resident_many_has(int kind, int rows, int strips, bool near) {
  if (rows != 2) return false;
  if (near) return strips == 1 || strips == 2 || (strips == 4 && kind != 1);
  return strips == (kind == 1 ? 2 : 4);
}

hipError_t launch_resident(int kind, int rows, int strips, bool near, const ResSolve& one, int n,
                           hipStream_t st) {
  const Kernel k = kernel_of(kind, rows, strips, near);
  if (!k || n < 1 || one.g.rows != rows || !one.sync || one.seq < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k, dim3(near ? 8 * n : n), dim3(kGroup), 0, st, one);
  return hipGetLastError();
}

hipError_t launch_resident_many(const ResSolve* many, const ResWg* wgs, int n, hipStream_t st) {
  if (n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_resident_many, dim3(n), dim3(kGroup), 0, st, many, wgs);
  return hipGetLastError();
}

hipError_t launch_resident_states(const ResSolve* many, int n, State* out, hipStream_t st) {
  if (n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_resident_states, dim3((n + 63) / 64), dim3(64), 0, st, many, n, out);
  return hipGetLastError();
}

size_t resident_area_bytes(int kind, const Geo& g, int strips) {
  const size_t nwg = (size_t)g.ntx * ((g.nty + strips - 1) / strips);
  const size_t nw = kind == 2 ? 1 : 2, cpl = kind == 2 ? 4 : 2;
  const size_t row = nw * cpl * kWave, col = nw * kResWaves * (size_t)g.rows * strips;
  return 8 * (kLine + (nwg + kLine - 1) / kLine * kLine + 2 * nwg * kLine + 4 * nwg * row +
              4 * nwg * col);
}

}  // namespace cgk
