// Fused WADG stage kernel for gfx950 for launches too small to fill the
// chip: a quarter of an element group (16 elements) per workgroup, each
// element spread over the four 16-lane subgroups of several waves.
//
// The same stage (or right-hand side, or the adjoint's apply-A products) and
// the same arithmetic as the other stage kernels (stage_common.h), every
// value by the same operations in the same order, so its results are bitwise
// theirs.  What such a launch costs is the time of one item, and with one
// element per lane that is one wave's chain of several hundred dependent
// operations behind 180 KB of loads by one CU.  Here lane (e, sub) of wave w
// does one short piece of element e's work in each phase:
//
//   A  wave 0: face sub (Section 6.4: traces, flux, lift); the other waves:
//      the point sums of quadrature column 4 (w - 1) + sub (Section 4.1), the
//      pressure columns first, then the velocity columns (a wave with both
//      kinds runs one after the other, as long as the face wave runs)
//   B  node row (field, b): the columns' sums and then the face terms added
//      to the row's load vector, and the row's part of the mass inverse
//      (rows in r of V_q Mhat^-1, Section 6.2)
//   C  inverse column (field, i): its points weighted by c^2/J or 1/J and
//      projected back in s
//   D  node row (field, b): projection in r and the update (Section 5.2)
//
// with the pieces' results exchanged through LDS (one barrier between
// phases).  The operators of the phases are the same for all lanes (scalar
// constants); only row i of V and D in phase A differs by lane.  Phases B to
// D deal their pieces to the waves from the last one on, because the face
// wave holds the most operands.
//
// A set has 1 + ceil(nq1 / 2) waves (Quarter::waves): 128 threads at nq1 = 2,
// 192 at 3 and 4, 256 at 5 and 6, 320 at 7.  Registers decide how many
// workgroups a CU holds: four of one wave per SIMD at N <= 3 (128 per lane),
// three at N = 4 (168).  FP64 instances that need more spill, and are used all
// the same where the measured time is shorter: stages at N = 3, nq1 = 4 (9
// registers) and 6 (63) and N = 4, nq1 = 6 (44), the apply-A + mass mode from
// N = 3 on (18 at nq1 = 5, 152 in the pair at nq1 = 6), sweeps of four sets from
// N = 2, nq1 = 5 on (40; 93 at N = 3, nq1 = 5; 177 at nq1 = 6), of three at N
// = 3, nq1 = 6 and N = 4 (24 to 99; 298 at nq1 = 7) and of two at N = 4, nq1 = 7
// (160).  No FP32 instance does.
//
// Measured on MI355X, one FP64 stage at N = 3, nq1 = 5 from a stream (an empty
// launch takes 2.4 us): 16 groups 8.3 -> 5.8 us against the split kernel's one
// item per workgroup, 64 groups 9.4 -> 6.9.
//
// quarter_sweep_kernel advances a whole slice of a mesh of few elements
// through all stages of many steps in one launch: the mesh is one workgroup
// (a set of these waves per 16 elements), the geometry stays in registers,
// the state in LDS and registers, and neighbour traces are read from LDS.
// Per stage on 16 elements: 7.9 -> 2.6 us with one slice, 61.6 -> 19.0 with
// 4096 (it reads and writes the state once per launch, and no lanes idle).

#include <hip/hip_runtime.h>

#include <type_traits>

#include "stage_common.h"

namespace wadg {
namespace {

using namespace dev;

constexpr int kQE = 16;      // elements per set

template <typename R, int N, int NQ>
struct Quarter {
  static constexpr int NP1 = N + 1, NP = NP1 * NP1, NQ2 = NQ * NQ;
  // Waves of a set: four at NQ = 5 and 6, one per SIMD (a fifth, as at NQ = 7,
  // shares SIMD 0 with the first in every workgroup, which then decides how
  // many workgroups a CU holds).
  static constexpr int waves = 1 + (2 * NQ + 3) / 4;
  static constexpr int pieces = 4 * waves;                     // per element and phase
  static_assert(pieces >= 3 * NP1, "one piece per node row");
  static_assert(2 * pieces >= 3 * NQ, "at most two inverse columns per piece");
  // LDS of a set, in values: the input tile [3][NP][16] (padded to whole 1 KB
  // rows of the copy), the inverses' values, the column sums (cr, cs, cx,
  // cy), the face terms, all in planes of 16.  In
  // the apply-A + mass mode the planes cr[a][b], cs[a][b] then hold the
  // pressure rows' factors of the sensitivity sum (read and rewritten by the
  // lanes of row b only).
  static constexpr unsigned row_planes = 64u / sizeof(R);      // planes of a 1 KB row
  static constexpr unsigned rows = (3u * NP + row_planes - 1) / row_planes;
  static constexpr unsigned tq = rows * 1024u / sizeof(R);
  // The planes are ordered so that the two subgroups of a half wave, which
  // access LDS together, find theirs an odd number of planes apart (16 FP64
  // values are half of the banks): strides over rows are odd, over columns
  // and faces one.
  static constexpr int st = 3 * NQ | 1, sc = NQ | 1, sf = 5;
  static constexpr unsigned xt = (unsigned)(st * NP1) * kQE;
  static constexpr unsigned xc = (unsigned)(4 * sc * NP1) * kQE;
  static constexpr unsigned xf = (unsigned)(3 * sf * NP1) * kQE;
  // inverse column q = c NQ + i, row b; sums k (cr, cs, cx, cy) of column i,
  // row b; face f, field c, face node (or row) m
  static __device__ constexpr int at_t(int q, int b) { return (b * st + q) * kQE; }
  static __device__ constexpr int at_c(int k, int i, int b) {
    return ((k * NP1 + b) * sc + i) * kQE;
  }
  static __device__ constexpr int at_f(int f, int c, int m) {
    return ((c * NP1 + m) * sf + f) * kQE;
  }
  static constexpr unsigned set = tq + xt + xc + xf;
  // sets of a workgroup that holds a whole mesh
  static constexpr int lds_sets = (int)(160u * 1024u / (set * sizeof(R)));
  static constexpr int max_sets = 16 / waves < lds_sets ? (16 / waves < 4 ? 16 / waves : 4)
                                                        : (lds_sets < 4 ? lds_sets : 4);
};

// One 1 KB row (64 lanes x 16 B) from global memory into LDS at dst, no
// registers; the caller waits (vmcnt) before the barrier that publishes it.
__device__ __forceinline__ void row_to_lds(rsrc_t src, void* dst, unsigned voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)dst, 16,
                                           voff, 0, 0, 0);
}

// The operators in memory, for phase A's lane-dependent rows.
template <typename R, int N, int NQ>
__device__ const ct::Ops<R, N, NQ> kOps = ct::make_ops<R, N, NQ>();

// What one lane holds and does.
template <typename R, int N, int NQ>
struct Lane {
  using L = Quarter<R, N, NQ>;
  static constexpr int NP1 = L::NP1, NP = L::NP;
  static constexpr unsigned KP = kWave * sizeof(R);

  int e, sub, w;            // element of the set, subgroup, wave of the set (uniform)
  unsigned kb;              // byte offset of the element's lane in a 64-lane plane
  R *tq, *xt, *xc, *xf;     // the set's LDS arrays

  // pieces of the phases: face or column i of phase A, row (c, b), inverse
  // column q; a column, row or inverse column that does not exist is computed
  // like the last one and not written
  int ia, c, b, row, piece;
  bool has_a, velocity, has_row;

  __device__ __forceinline__ Lane(int e_, int sub_, int w_, int e0, R* lds)
      : e(e_), sub(sub_), w(w_), kb((unsigned)(e0 + e_) * (unsigned)sizeof(R)), tq(lds),
        xt(lds + L::tq), xc(lds + L::tq + L::xt), xf(lds + L::tq + L::xt + L::xc) {
    const int col = 4 * (w - 1) + sub;                         // phase A, w > 0
    velocity = col >= NQ;
    has_a = col < 2 * NQ;
    ia = w == 0 ? sub : has_a ? col - (velocity ? NQ : 0) : NQ - 1;
    piece = 4 * (L::waves - 1 - w) + sub;                      // phases B to D
    has_row = piece < 3 * NP1;
    row = has_row ? piece : 3 * NP1 - 1;
    c = row / NP1;
    b = row - c * NP1;
  }
  // byte offset of node a of the lane's row in a tiled state
  __device__ __forceinline__ unsigned rowoff() const {
    return kb + (unsigned)(c * NP + NP1 * b) * KP;
  }

  // Phase B, first part: the load vector of the lane's row, volume term then
  // face terms in face order 0..3 (faces 0 and 2 are the rows b = 0 and N,
  // faces 3 and 1 the first and last node of every row).
  __device__ __forceinline__ void load_vector(R (&v)[NP1]) const {
#pragma unroll
    for (int a = 0; a < NP1; ++a) v[a] = R(0);
    if (c == 0) {
#pragma unroll
      for (int i = 0; i < NQ; ++i)
        pressure_column_add<R, N, NQ>(i, xc[L::at_c(0, i, b) + e],
                                      xc[L::at_c(1, i, b) + e], v);
    } else {
#pragma unroll
      for (int i = 0; i < NQ; ++i)
        velocity_column_add<R, N, NQ>(i, xc[L::at_c(1 + c, i, b) + e], v);
    }
    if (b == 0) {
#pragma unroll
      for (int m = 0; m < NP1; ++m) v[m] += xf[L::at_f(0, c, m) + e];
    }
    v[N] += xf[L::at_f(1, c, b) + e];
    if (b == N) {
#pragma unroll
      for (int m = 0; m < NP1; ++m) v[m] += xf[L::at_f(2, c, m) + e];
    }
    v[0] += xf[L::at_f(3, c, b) + e];
  }
  // Phase B, second part: the row of the mass inverse in r.
  __device__ __forceinline__ void inverse_row(const R (&r)[NP1]) {
    constexpr ct::Ops<R, N, NQ> T = ct::make_ops<R, N, NQ>();
    if (!has_row) return;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      R t = R(0);
#pragma unroll
      for (int a = 0; a < NP1; ++a) t = mad(T.Vt[i][a], r[a], t);
      xt[L::at_t(c * NQ + i, b) + e] = t;
    }
  }
  // Phase D: projection of the lane's row in r.
  __device__ __forceinline__ void project_row(R (&dq)[NP1]) const {
    constexpr ct::Ops<R, N, NQ> T = ct::make_ops<R, N, NQ>();
#pragma unroll
    for (int a = 0; a < NP1; ++a) dq[a] = R(0);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const R s = xt[L::at_t(c * NQ + i, b) + e];
#pragma unroll
      for (int a = 0; a < NP1; ++a) dq[a] = mad(T.P[a][i], s, dq[a]);
    }
  }
};

// Phase C's piece: inverse column q = c NQ + i, with its mass weights held
// (scaled by c2_scale for the pressure, as every kernel forms them).
template <typename R, int N, int NQ>
struct InverseColumn {
  using L = Quarter<R, N, NQ>;
  static constexpr int NP1 = L::NP1;
  static constexpr unsigned KP = kWave * sizeof(R);
  int q;
  bool exists;
  R w[NQ];

  __device__ __forceinline__ void load(const Lane<R, N, NQ>& ln, int piece, rsrc_t vol) {
    exists = piece < 3 * NQ;
    q = exists ? piece : 3 * NQ - 1;
    const int c = q / NQ;
    const unsigned o = ln.kb + (unsigned)((c == 0 ? 4 : 5) * NQ * NQ + q - c * NQ) * KP;
#pragma unroll
    for (int j = 0; j < NQ; ++j) w[j] = ldr<R>(vol, o, NQ * j * KP);
  }
  __device__ __forceinline__ void scale(R c2s) {
    if (q < NQ) {
#pragma unroll
      for (int j = 0; j < NQ; ++j) w[j] *= c2s;
    }
  }
  __device__ __forceinline__ void run(const Lane<R, N, NQ>& ln) const {
    constexpr ct::Ops<R, N, NQ> T = ct::make_ops<R, N, NQ>();
    R t[NP1], s[NP1];
#pragma unroll
    for (int m = 0; m < NP1; ++m) {
      t[m] = ln.xt[L::at_t(q, m) + ln.e];
      s[m] = R(0);
    }
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      R rq = R(0);
#pragma unroll
      for (int m = 0; m < NP1; ++m) rq = mad(T.Vt[j][m], t[m], rq);
      rq *= w[j];
#pragma unroll
      for (int m = 0; m < NP1; ++m) s[m] = mad(T.P[m][j], rq, s[m]);
    }
    if (exists) {
#pragma unroll
      for (int m = 0; m < NP1; ++m) ln.xt[L::at_t(q, m) + ln.e] = s[m];
    }
  }
};

// Phase C of a lane: its inverse column, and in the first waves a second one
// where there are more columns than pieces.
template <typename R, int N, int NQ>
struct InverseColumns {
  using L = Quarter<R, N, NQ>;
  static constexpr bool kTwo = 3 * NQ > L::pieces;
  InverseColumn<R, N, NQ> a, b;
  __device__ __forceinline__ static bool second(const Lane<R, N, NQ>& ln) {
    return kTwo && 4 * (L::waves - 1 - ln.w) + L::pieces < 3 * NQ;   // wave-uniform
  }
  __device__ __forceinline__ void load(const Lane<R, N, NQ>& ln, rsrc_t vol) {
    a.load(ln, ln.piece, vol);
    if constexpr (kTwo) {
      if (second(ln)) b.load(ln, ln.piece + L::pieces, vol);
    }
  }
  __device__ __forceinline__ void scale(const Lane<R, N, NQ>& ln, R c2s) {
    a.scale(c2s);
    if constexpr (kTwo) {
      if (second(ln)) b.scale(c2s);
    }
  }
  __device__ __forceinline__ void run(const Lane<R, N, NQ>& ln) const {
    a.run(ln);
    if constexpr (kTwo) {
      if (second(ln)) b.run(ln);
    }
  }
};

// Phase A's work of a wave, by its role, with the operands held for it:
// faces, or columns of the pressure or the velocity alone or of both.
enum Role { kFace, kPressure, kVelocity, kBoth };

template <typename R, int N, int NQ, int ROLE>
struct Piece {
  using L = Quarter<R, N, NQ>;
  static constexpr int NP1 = L::NP1, NP = L::NP;
  static constexpr unsigned KP = kWave * sizeof(R);
  R g[4][NQ], vi[NP1], di[NP1];

  __device__ __forceinline__ void load(const Lane<R, N, NQ>& ln, rsrc_t vol, rsrc_t face) {
    if constexpr (ROLE == kFace) {
      const unsigned o = ln.kb + (unsigned)(ln.ia * NQ) * KP;
#pragma unroll
      for (int cc = 0; cc < 3; ++cc)
#pragma unroll
        for (int j = 0; j < NQ; ++j) g[cc][j] = ldr<R>(face, o, (cc * 4 * NQ + j) * KP);
    } else {
      const unsigned o = ln.kb + (unsigned)ln.ia * KP;
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < NQ; ++j) g[q][j] = ldr<R>(vol, o, (q * NQ * NQ + NQ * j) * KP);
#pragma unroll
      for (int a = 0; a < NP1; ++a) {
        vi[a] = kOps<R, N, NQ>.V[ln.ia][a];
        di[a] = kOps<R, N, NQ>.D[ln.ia][a];
      }
    }
  }
  // Face of the lane (node m of face f is f0 + fs m).
  __device__ __forceinline__ void face(const Lane<R, N, NQ>& ln, const StageScalars<R>& k,
                                       const Trace<R, N>& tr) const {
    const int f = ln.ia, e = ln.e;
    const R* t = ln.tq + ((f == 1 ? N : f == 2 ? N * NP1 : 0) * kQE + e);
    const int fs = ((f & 1) ? NP1 : 1) * kQE;
    auto P = [&](int m) { return t[fs * m]; };
    auto U = [&](int m) { return t[NP * kQE + fs * m]; };
    auto V = [&](int m) { return t[2 * NP * kQE + fs * m]; };
    R gf[3][NQ];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc)
#pragma unroll
      for (int j = 0; j < NQ; ++j) gf[cc][j] = g[cc][j];
    R sp[NP1], su[NP1], sv[NP1];
    face_terms<R, N, NQ, true, true>(0, P, U, V, tr, gf, k.tau_p, k.tau_u, sp, su, sv);
#pragma unroll
    for (int m = 0; m < NP1; ++m) {
      ln.xf[L::at_f(f, 0, m) + e] = sp[m];
      ln.xf[L::at_f(f, 1, m) + e] = su[m];
      ln.xf[L::at_f(f, 2, m) + e] = sv[m];
    }
  }
  // Sums of the lane's column over its points.
  template <bool PRESSURE>
  __device__ __forceinline__ void column_of(const Lane<R, N, NQ>& ln) const {
    const int e = ln.e;
    auto P = [&](int n) { return ln.tq[n * kQE + e]; };
    auto U = [&](int n) { return ln.tq[(NP + n) * kQE + e]; };
    auto V = [&](int n) { return ln.tq[(2 * NP + n) * kQE + e]; };
    R c0[NP1], c1[NP1];
    if constexpr (PRESSURE)
      pressure_column_sums<R, N, NQ, true>(vi, U, V, g, c0, c1);
    else
      velocity_column_sums<R, N, NQ, true>(vi, di, P, g, c0, c1);
    if (ln.has_a) {
      constexpr int q = PRESSURE ? 0 : 2;
#pragma unroll
      for (int m = 0; m < NP1; ++m) {
        ln.xc[L::at_c(q, ln.ia, m) + e] = c0[m];
        ln.xc[L::at_c(q + 1, ln.ia, m) + e] = c1[m];
      }
    }
  }
  __device__ __forceinline__ void column(const Lane<R, N, NQ>& ln) const {
    if constexpr (ROLE == kPressure) {
      column_of<true>(ln);
    } else if constexpr (ROLE == kVelocity) {
      column_of<false>(ln);
    } else {
      if (!ln.velocity) column_of<true>(ln);
      if (ln.velocity) column_of<false>(ln);
    }
  }
};

// f(role) for wave w of a set.
template <int NQ, typename F>
__device__ __forceinline__ void by_role(int w, const F& f) {
  if (w == 0)
    f(std::integral_constant<int, kFace>{});
  else if (4 * w <= NQ)
    f(std::integral_constant<int, kPressure>{});
  else if (4 * (w - 1) >= NQ)
    f(std::integral_constant<int, kVelocity>{});
  else
    f(std::integral_constant<int, kBoth>{});
}

// Workgroup bid of a launch of nb workgroups over the slices' 16-element sets.
template <typename R, int N, int NQ, int MODE>
__device__ __forceinline__ void quarter_run(const StageParams& p, int bid, int nb, R* lds) {
  static_assert((MODE != kApplyA && MODE != kApplyAMass) || sizeof(R) == sizeof(double),
                "apply-A modes are FP64 only");
  using L = Quarter<R, N, NQ>;
  constexpr int NP1 = L::NP1, NP = L::NP;
  constexpr unsigned tile = 3u * NP * kWave;
  constexpr unsigned tb = tile * sizeof(R);
  constexpr unsigned KP = kWave * sizeof(R);
  constexpr bool kMass = MODE == kApplyAMass;
  const int nset = (p.K + kQE - 1) / kQE;
  int s, qs;
  item_coords(item_of(bid, nb, p.reverse), nset, p.S, min(4 * p.tile_groups, nset), p.tile_slices,
              s, qs);
  const int eg = qs >> 2, e0 = (qs & 3) * kQE;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Lane<R, N, NQ> ln(lane & (kQE - 1), lane / kQE, wave, e0, lds);
  const bool active = eg * kWave + e0 + ln.e < p.K;
  const StageScalars<R> k = stage_scalars<R>(p);

  const R* Qin = static_cast<const R*>(p.Qin);
  const size_t slice = (size_t)s * p.nEG * tile;
  const size_t grp = slice + (size_t)eg * tile;
  const rsrc_t vol = make_rsrc(static_cast<const R*>(p.vol) + (size_t)eg * 6 * L::NQ2 * kWave,
                               6u * L::NQ2 * KP);

  const rsrc_t face = make_rsrc(static_cast<const R*>(p.face) + (size_t)eg * 12 * NQ * kWave,
                                12u * NQ * KP);
  const unsigned ro = ln.rowoff();
  R resv[NP1], rb[NP1], ri[NP1], rp[NP1], q[NP1];
  InverseColumns<R, N, NQ> inv;
#pragma unroll
  for (int a = 0; a < NP1; ++a) resv[a] = R(0);
  // the operands of the later phases
  auto late_loads = [&](auto with_rows) {
    constexpr bool kRows = decltype(with_rows)::value;
    if constexpr (kRows && MODE != kRhs) {
      if (MODE != kStage || k.A != R(0)) {
        const rsrc_t res = make_rsrc(static_cast<const R*>(p.res) + grp, tb);
#pragma unroll
        for (int a = 0; a < NP1; ++a) resv[a] = ldr<R>(res, ro, a * KP);
      }
    }
    if constexpr (kRows && kMass) {
      // absent operands read as zeros through empty resources; the pressure
      // rows alone use r_i and r_{i-1}
      const AdjMassParams& am = p.adj;
      const rsrc_t rbr = make_rsrc(am.rbar + grp, am.a_next != 0.0 ? tb : 0u);
      const rsrc_t rir = make_rsrc(am.r + grp, NP * KP);
      const rsrc_t rpr = make_rsrc(am.r_prev ? am.r_prev + grp : am.r + grp,
                                   (am.a != 0.0 && am.r_prev) ? NP * KP : 0u);
#pragma unroll
      for (int a = 0; a < NP1; ++a) {
        rb[a] = ldr<R>(rbr, ro, a * KP);
        ri[a] = ldr<R>(rir, ro, a * KP);
        rp[a] = ldr<R>(rpr, ro, a * KP);
      }
    }
    if constexpr (MODE != kApplyA) inv.load(ln, vol);
  };
  by_role<NQ>(wave, [&](auto role) {
    constexpr int ROLE = decltype(role)::value;
    Piece<R, N, NQ, ROLE> pc;
    Trace<R, N> tr;
    using Rows = std::integral_constant<bool, ROLE != kFace || (L::pieces - 4 < 3 * NP1)>;
    // loads: the set's part of the input tile into LDS (16 B per lane, one
    // plane in sizeof(R) lanes) by the waves without faces, whose traces are
    // a chain of two loads; then every lane's operands
    if constexpr (ROLE == kFace) {
      const rsrc_t nbr = make_rsrc(p.nbr + (size_t)eg * 8 * kWave, 8u * kWave * 4u);
      const unsigned no = (unsigned)(e0 + ln.e + ln.ia * kWave) * 4u;
      const unsigned base = (unsigned)ldi(nbr, no, 0);
      const int step = ldi(nbr, no, 4 * kWave * 4);
      pc.load(ln, vol, face);
      const rsrc_t qslice = make_rsrc(Qin + slice, (unsigned)p.nEG * tb);
#pragma unroll
      for (int m = 0; m < NP1; ++m) {
        const unsigned off = (base + (unsigned)(step * m)) * (unsigned)sizeof(R);
        tr.p[m] = ldr<R>(qslice, off, 0);
        tr.u[m] = ldr<R>(qslice, off, NP * KP);
        tr.v[m] = ldr<R>(qslice, off, 2 * NP * KP);
      }
      late_loads(Rows{});
    } else {
      const rsrc_t qin = make_rsrc(Qin + grp, tb);
      constexpr unsigned lpp = sizeof(R);                      // lanes of a plane's 16 elements
      const unsigned lo = ((unsigned)lane / lpp) * KP + ((unsigned)lane % lpp) * 16u + e0 * lpp;
      for (unsigned r = (unsigned)wave - 1u; r < L::rows; r += L::waves - 1)
        row_to_lds(qin, reinterpret_cast<char*>(lds) + r * 1024u, r * L::row_planes * KP + lo);
      pc.load(ln, vol, face);
      late_loads(Rows{});
      __builtin_amdgcn_s_waitcnt(0x0F70);                      // the tile's rows (vmcnt = 0)
    }
    __syncthreads();                                           // tile in LDS
    if constexpr (Rows::value && MODE == kStage) {             // the row's input values
#pragma unroll
      for (int a = 0; a < NP1; ++a) q[a] = ln.tq[(ln.row * NP1 + a) * kQE + ln.e];
    }
    if constexpr (ROLE == kFace)
      pc.face(ln, k, tr);
    else
      pc.column(ln);
  });
  __syncthreads();                                             // column sums, face terms

  const rsrc_t qout = make_rsrc(static_cast<R*>(p.Qout) + grp, tb);
  const bool write = active && ln.has_row;
  R v[NP1];
  ln.load_vector(v);
  if constexpr (MODE == kApplyA || kMass) {
    // ybar + dt D A z; the mass step of the next reverse stage follows on it
    const R sdt = ln.c == 0 ? k.dt : -k.dt;
#pragma unroll
    for (int a = 0; a < NP1; ++a) v[a] = mad(sdt, v[a], resv[a]);
    if (write) {
#pragma unroll
      for (int a = 0; a < NP1; ++a) st(qout, ro, a * KP, v[a]);
    }
  }
  if constexpr (MODE == kApplyA) return;
  if constexpr (kMass) {
    const AdjMassParams& am = p.adj;
#pragma unroll
    for (int a = 0; a < NP1; ++a) v[a] = mad(R(am.a_next), rb[a], R(am.b) * v[a]);
    if (ln.c == 0) {
#pragma unroll
      for (int a = 0; a < NP1; ++a) {
        ln.xc[L::at_c(0, a, ln.b) + ln.e] = v[a];
        ln.xc[L::at_c(1, a, ln.b) + ln.e] = mad(R(-am.a), rp[a], ri[a]);
      }
    }
    if (write) {
      const rsrc_t rbw = make_rsrc(am.rbar + grp, tb);
#pragma unroll
      for (int a = 0; a < NP1; ++a) st(rbw, ro, a * KP, v[a]);
    }
  }
  ln.inverse_row(v);
  __syncthreads();                                             // rows of the inverse
  inv.scale(ln, k.c2s);
  inv.run(ln);
  if constexpr (kMass) {
    // sum over the pressure values of rbar (r_i - A_i r_{i-1}), node order
    if (ln.w == 0 && ln.sub == 0) {
      R dot = R(0);
#pragma unroll
      for (int n = 0; n < NP; ++n)
        dot = mad(ln.xc[L::at_c(0, n % NP1, n / NP1) + ln.e],
                  ln.xc[L::at_c(1, n % NP1, n / NP1) + ln.e], dot);
      if (!active) dot = R(0);
      dot = sum16(dot);
      if (ln.e == 0) p.adj.part[4 * (s * p.nEG + eg) + (qs & 3)] += dot;
    }
  }
  __syncthreads();                                             // columns projected in s
  R dq[NP1];
  ln.project_row(dq);
  if (!write) return;
  if constexpr (MODE == kRhs) {
#pragma unroll
    for (int a = 0; a < NP1; ++a) st(qout, ro, a * KP, dq[a]);
  } else if constexpr (kMass) {
    const rsrc_t zo = make_rsrc(p.adj.z + grp, tb);
    const R sg = ln.c == 0 ? R(1) : R(-1);
#pragma unroll
    for (int a = 0; a < NP1; ++a) st(zo, ro, a * KP, sg * dq[a]);
  } else {
    const rsrc_t resw = make_rsrc(static_cast<R*>(p.res_out ? p.res_out : p.res) + grp,
                                  p.res_dead ? 0u : tb);
#pragma unroll
    for (int a = 0; a < NP1; ++a) {
      const R r = mad(k.A, resv[a], k.dt * dq[a]);
      st(resw, ro, a * KP, r);
      st(qout, ro, a * KP, mad(k.B, r, q[a]));
    }
  }
}

}  // namespace

template <typename R, int N, int NQ, int MODE>
__global__ __launch_bounds__((Quarter<R, N, NQ>::waves * kWave),
                             N <= 3 ? 4 : 3) void quarter_kernel(const StageParams p) {
  __shared__ __attribute__((aligned(1024))) R lds[Quarter<R, N, NQ>::set];
  quarter_run<R, N, NQ, MODE>(p, blockIdx.x, gridDim.x, lds);
}

// Two independent launches in one grid (FP64), as split_pair_kernel: the
// sets of launch a in mode MA (an apply-A mode), then the LSRK stage sets of
// launch b.
template <typename R, int N, int NQ, int MA>
__global__ __launch_bounds__((Quarter<R, N, NQ>::waves * kWave),
                             N <= 3 ? 4 : 3) void quarter_pair_kernel(const StageParams a,
                                                                     const StageParams b, int na) {
  __shared__ __attribute__((aligned(1024))) R lds[Quarter<R, N, NQ>::set];
  if ((int)blockIdx.x < na)
    quarter_run<R, N, NQ, MA>(a, blockIdx.x, na, lds);
  else
    quarter_run<R, N, NQ, kStage>(b, blockIdx.x - na, gridDim.x - na, lds);
}

// Whole sweep of slice blockIdx.x of a mesh of one element group and at most
// 16 SETS elements: nsteps steps from Qin to Qout (FP64, may be the same; R
// inside).
template <typename R, int N, int NQ, int SETS>
__global__ __launch_bounds__((SETS * Quarter<R, N, NQ>::waves * kWave)) void quarter_sweep_kernel(
    const double* Qin, double* Qout, const StageParams p, const SweepCoefs rk, int nsteps) {
  using L = Quarter<R, N, NQ>;
  constexpr int NP1 = L::NP1, NP = L::NP;
  constexpr unsigned tile = 3u * NP * kWave;
  constexpr unsigned KP = kWave * sizeof(R);
  __shared__ __attribute__((aligned(1024))) R lds[SETS * L::set];
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = wave / L::waves;
  Lane<R, N, NQ> ln(lane & (kQE - 1), lane / kQE, wave - set * L::waves, set * kQE,
                    lds + (size_t)set * L::set);
  const bool active = set * kQE + ln.e < p.K;
  const StageScalars<R> k = stage_scalars<R>(p);

  const rsrc_t vol = make_rsrc(p.vol, 6u * L::NQ2 * KP);
  const rsrc_t face = make_rsrc(p.face, 12u * NQ * KP);
  const size_t mine = (size_t)blockIdx.x * tile + (size_t)ln.row * NP1 * kWave + set * kQE + ln.e;
  by_role<NQ>(wave - set * L::waves, [&](auto role) {
    constexpr int ROLE = decltype(role)::value;
    Piece<R, N, NQ, ROLE> pc;
    pc.load(ln, vol, face);
    const R* nb = lds;             // the neighbour's value at my face node 0, and the step
    int ns = 0;
    if constexpr (ROLE == kFace) {
      const rsrc_t nbr = make_rsrc(p.nbr, 8u * kWave * 4u);
      const unsigned no = (unsigned)(set * kQE + ln.e + ln.ia * kWave) * 4u;
      const int base = ldi(nbr, no, 0), step = ldi(nbr, no, 4 * kWave * 4);
      if (active) {                // (padding lanes have no neighbour)
        const int k2 = base & (kWave - 1);
        nb = lds + ((k2 / kQE) * (int)L::set + (base / kWave) * kQE + (k2 & (kQE - 1)));
        ns = step / (kWave / kQE);
      }
    }
    InverseColumns<R, N, NQ> inv;
    inv.load(ln, vol);
    inv.scale(ln, k.c2s);
    R q[NP1], resv[NP1];
#pragma unroll
    for (int a = 0; a < NP1; ++a) q[a] = (R)Qin[mine + a * kWave];
    auto publish = [&] {
      if (ln.has_row) {
#pragma unroll
        for (int a = 0; a < NP1; ++a) ln.tq[(ln.row * NP1 + a) * kQE + ln.e] = q[a];
      }
    };
    publish();
    for (int stp = 0; stp < nsteps; ++stp) {
#pragma unroll
      for (int a = 0; a < NP1; ++a) resv[a] = R(0);
#pragma unroll 1
      for (int i = 0; i < 5; ++i) {
        const R rkA = (R)rk.A[i], rkB = (R)rk.B[i];
        __syncthreads();                                       // tile in LDS
        if constexpr (ROLE == kFace) {
          Trace<R, N> tr;
#pragma unroll
          for (int m = 0; m < NP1; ++m) {
            tr.p[m] = nb[ns * m];
            tr.u[m] = nb[ns * m + NP * kQE];
            tr.v[m] = nb[ns * m + 2 * NP * kQE];
          }
          pc.face(ln, k, tr);
        } else {
          pc.column(ln);
        }
        __syncthreads();                                       // column sums, face terms
        R v[NP1];
        ln.load_vector(v);
        ln.inverse_row(v);
        __syncthreads();                                       // rows of the inverse
        inv.run(ln);
        __syncthreads();                                       // columns projected in s
        R dq[NP1];
        ln.project_row(dq);
#pragma unroll
        for (int a = 0; a < NP1; ++a) {
          resv[a] = mad(rkA, resv[a], k.dt * dq[a]);
          q[a] = mad(rkB, resv[a], q[a]);
        }
        publish();
      }
    }
    if (active && ln.has_row) {
#pragma unroll
      for (int a = 0; a < NP1; ++a) Qout[mine + a * kWave] = (double)q[a];
    }
  });
}

namespace {

int64_t sets_of(const StageParams& p) { return (int64_t)((p.K + kQE - 1) / kQE) * p.S; }

template <typename R, int N, int NQ>
int launch_nq(int mode, const StageParams& p, void* stream) {
  const dim3 grid((unsigned)sets_of(p)), block(Quarter<R, N, NQ>::waves * kWave);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (mode == kStage) {
    hipLaunchKernelGGL((quarter_kernel<R, N, NQ, kStage>), grid, block, 0, st, p);
  } else if constexpr (sizeof(R) == sizeof(double)) {
    if (mode == kRhs)
      hipLaunchKernelGGL((quarter_kernel<R, N, NQ, kRhs>), grid, block, 0, st, p);
    else if (mode == kApplyA)
      hipLaunchKernelGGL((quarter_kernel<R, N, NQ, kApplyA>), grid, block, 0, st, p);
    else if (mode == kApplyAMass)
      hipLaunchKernelGGL((quarter_kernel<R, N, NQ, kApplyAMass>), grid, block, 0, st, p);
    else
      return (int)hipErrorInvalidValue;
  } else {
    return (int)hipErrorInvalidValue;
  }
  return (int)hipGetLastError();
}

template <int N, int NQ>
int launch_pair_nq(int mode_a, const StageParams& a, const StageParams& b, void* stream) {
  const int na = (int)sets_of(a), nb = (int)sets_of(b);
  const dim3 grid(na + nb), block(Quarter<double, N, NQ>::waves * kWave);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (mode_a == kApplyAMass)
    hipLaunchKernelGGL((quarter_pair_kernel<double, N, NQ, kApplyAMass>), grid, block, 0, st, a, b,
                       na);
  else if (mode_a == kApplyA)
    hipLaunchKernelGGL((quarter_pair_kernel<double, N, NQ, kApplyA>), grid, block, 0, st, a, b, na);
  else
    return (int)hipErrorInvalidValue;
  return (int)hipGetLastError();
}

template <typename R, int N, int NQ, int SETS = 1>
int launch_sweep_nq(const double* Qin, double* Qout, const StageParams& p, const SweepCoefs& rk,
                    int nsteps, void* stream) {
  using L = Quarter<R, N, NQ>;
  if constexpr (SETS <= L::max_sets) {
    if (p.K > SETS * kQE)
      return launch_sweep_nq<R, N, NQ, SETS + 1>(Qin, Qout, p, rk, nsteps, stream);
    // (HIP takes fewer than 2^32 lanes per launch: 11 million slices at six waves)
    constexpr int threads = SETS * L::waves * kWave;
    constexpr int64_t most = ((1LL << 32) - 1) / threads;
    constexpr size_t tile = (size_t)3 * L::NP * kWave;
    for (int64_t s0 = 0; s0 < p.S; s0 += most) {
      hipLaunchKernelGGL((quarter_sweep_kernel<R, N, NQ, SETS>),
                         dim3((unsigned)(p.S - s0 < most ? p.S - s0 : most)), dim3(threads), 0,
                         static_cast<hipStream_t>(stream), Qin + s0 * tile, Qout + s0 * tile, p, rk,
                         nsteps);
      const int e = (int)hipGetLastError();
      if (e) return e;
    }
    return 0;
  } else {
    return (int)hipErrorInvalidValue;
  }
}

// The launches of a degree and quadrature, by (N, nq - N).
template <int N, int NQ>
struct Launch {
  static int stage(int mode, const StageParams& p, void* stream) {
    return launch_nq<double, N, NQ>(mode, p, stream);
  }
  static int stage_fp32(int mode, const StageParams& p, void* stream) {
    return launch_nq<float, N, NQ>(mode, p, stream);
  }
  static int pair(int mode_a, const StageParams& a, const StageParams& b, void* stream) {
    return launch_pair_nq<N, NQ>(mode_a, a, b, stream);
  }
  static int elements(bool fp32) {
    return kQE * (fp32 ? Quarter<float, N, NQ>::max_sets : Quarter<double, N, NQ>::max_sets);
  }
  static int sweep(const double* Qin, double* Qout, const StageParams& p, const SweepCoefs& rk,
                   int nsteps, bool fp32, void* stream) {
    return fp32 ? launch_sweep_nq<float, N, NQ>(Qin, Qout, p, rk, nsteps, stream)
                : launch_sweep_nq<double, N, NQ>(Qin, Qout, p, rk, nsteps, stream);
  }
};

struct LaunchTable {
  decltype(&Launch<1, 2>::stage) stage, stage_fp32;
  decltype(&Launch<1, 2>::pair) pair;
  decltype(&Launch<1, 2>::elements) elements;
  decltype(&Launch<1, 2>::sweep) sweep;
};

template <int N, int NQ>
constexpr LaunchTable entry() {
  using L = Launch<N, NQ>;
  return {&L::stage, &L::stage_fp32, &L::pair, &L::elements, &L::sweep};
}

const LaunchTable* table(int N, int nq) {
  static const LaunchTable t[4][3] = {{entry<1, 2>(), entry<1, 3>(), entry<1, 4>()},
                                      {entry<2, 3>(), entry<2, 4>(), entry<2, 5>()},
                                      {entry<3, 4>(), entry<3, 5>(), entry<3, 6>()},
                                      {entry<4, 5>(), entry<4, 6>(), entry<4, 7>()}};
  return stage_supported(N, nq) ? &t[N - 1][nq - N - 1] : nullptr;
}

}  // namespace

int launch_stage_quarter(int N, int nq, int mode, const StageParams& p, void* stream) {
  const LaunchTable* t = table(N, nq);
  if (!t || sets_of(p) >= (1LL << 31)) return (int)hipErrorInvalidValue;
  return t->stage(mode, p, stream);
}

int launch_stage_quarter_fp32(int N, int nq, const StageParams& p, void* stream) {
  const LaunchTable* t = table(N, nq);
  if (!t || sets_of(p) >= (1LL << 31)) return (int)hipErrorInvalidValue;
  return t->stage_fp32(kStage, p, stream);
}

int launch_stage_quarter_pair(int N, int nq, int mode_a, const StageParams& a,
                              const StageParams& b, void* stream) {
  const LaunchTable* t = table(N, nq);
  if (!t || sets_of(a) + sets_of(b) >= (1LL << 31)) return (int)hipErrorInvalidValue;
  return t->pair(mode_a, a, b, stream);
}

int quarter_sweep_elements(int N, int nq, bool fp32) {
  const LaunchTable* t = table(N, nq);
  return t ? t->elements(fp32) : 0;
}

int launch_sweep_quarter(int N, int nq, const double* Qin, double* Qout, const StageParams& p,
                         const SweepCoefs& rk, int nsteps, bool fp32, void* stream) {
  const LaunchTable* t = table(N, nq);
  if (!t) return (int)hipErrorInvalidValue;
  return t->sweep(Qin, Qout, p, rk, nsteps, fp32, stream);
}

}  // namespace wadg
