// The smooth solve, the Newton solve and the implicit velocity update with one dof per lane
// and the matrices' rows in registers (mjh_lanes.h), for worlds of at most 28 dofs that fit
// their team and whose contacts are all condim-3 pyramids (DevModel::jframe).  The
// mathematics is newton_impl's; what differs is where things live:
//   - row i of M, then of the Newton Hessian H and of its inverse, are in lane i's registers;
//   - a contact's four edge rows are on the four lanes of a quad (lane r of a chunk of T rows
//     holds edge r), so that the edges J_n +- mu J_tk of a product come from the frame rows'
//     products by quad permutations;
//   - H is summed on the matrix cores, a contraction over the frame rows, and eliminated there
//     too (SymAcc; 32-lane teams: two worlds at once, one 32 x 32 block each);
//   - limit and friction-loss rows are unit vectors: they add to one dof's gradient and to
//     one diagonal entry;
//   - control flow is uniform in the wavefront and every lane is active: a team that is done
//     runs along without updating, because matrix instructions and lane swaps take all lanes.
// The solves in LDS were bound by their serial chains: every entry of a triangular solve and
// every four columns of a factor waited for an LDS or readlane round trip, and packed indices
// were unranked per entry.  Measured against them, before the other phases changed: 8192
// quadrupeds x 3 steps 662 -> 323 us, 64 x 4 steps 530 -> 204 us, 2048 humanoids x 2 steps 491 ->
// 200 us, 8192 hands x 4 steps 2079 -> 1120 us; with them as they are now 248, 142, 140 and 645.
#pragma once

namespace mjh {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// the largest of the wavefront's teams' values, as a scalar
template <int T>
DEV int wave_max(int v) {
  int r = __builtin_amdgcn_readlane(v, 0);
  if constexpr (T <= 32) r = max(r, __builtin_amdgcn_readlane(v, 32));
  if constexpr (T == 16)
    r = max(r, max(__builtin_amdgcn_readlane(v, 16), __builtin_amdgcn_readlane(v, 48)));
  return r;
}
// whether some lane of this team has the flag set
template <int T>
DEV bool team_any(bool f, int lane) {
  const unsigned long long b = __ballot(f);
  if constexpr (T == 64) return b != 0;
  const int base = (int)(threadIdx.x & 63) - lane;
  return ((b >> base) & ((1ull << (T & 63)) - 1ull)) != 0;
}
// sum over the dofs (a 64-lane team holds each twice)
template <int T>
DEV float dof_sum(const Team& t, float v) {
  return Team{t.lane, T == 16 ? 16 : 32, t.tp}.sum(v);
}
template <int T>
DEV float dof_max(const Team& t, float v) {
  return Team{t.lane, T == 16 ? 16 : 32, t.tp}.max(v);
}

// Two reductions at once, by row and by dof: the wider steps come first and fold the two values
// onto different rows (or halves), so that the steps within a row are shared.  A Newton iteration
// has four such pairs, each a chain of 60 to 80 clocks: 65536 quadrupeds 415 -> 407 us, 8192 x 3
// 254 -> 248, 2048 humanoids x 2 155 -> 140.
template <class Op>
DEV float row_reduce(float v, Op op) {  // over a 16-lane row
  v = op(v, quad_perm<kXor1>(v));
  v = op(v, quad_perm<kXor2>(v));
  v = op(v, quad_perm<0x141>(v));  // row_half_mirror
  return op(v, quad_perm<0x140>(v));  // row_mirror
}
template <class Op>
DEV Pair reduce2_32(float x, float y, Op op) {  // over each half-wavefront
  const auto h = __builtin_amdgcn_permlane16_swap((unsigned)__float_as_int(x),
                                                  (unsigned)__float_as_int(y), false, false);
  return swap16(row_reduce(op(__int_as_float((int)h[0]), __int_as_float((int)h[1])), op));
}
template <int T, class Op>
DEV Pair reduce2(float x, float y, Op op) {
  if constexpr (T == 16) return {row_reduce(x, op), row_reduce(y, op)};
  if constexpr (T == 32) return reduce2_32(x, y, op);
  const Pair h = swap32(x, y);
  const float v = row_reduce(op(h.a, h.b), op);
  const Pair w = swap16(v);
  const float r = op(w.a, w.b);
  return swap32(r, r);
}
struct OpAdd { DEV float operator()(float a, float b) const { return a + b; } };
struct OpMax { DEV float operator()(float a, float b) const { return fmaxf(a, b); } };
template <int T>
DEV Pair sum2(float x, float y) { return reduce2<T>(x, y, OpAdd()); }
template <int T>
DEV Pair max2(float x, float y) { return reduce2<T>(x, y, OpMax()); }
// (a 64-lane team holds every dof on both halves)
template <int T>
DEV Pair dof_sum2(float x, float y) { return reduce2<T == 16 ? 16 : 32>(x, y, OpAdd()); }
template <int T>
DEV Pair dof_max2(float x, float y) { return reduce2<T == 16 ? 16 : 32>(x, y, OpMax()); }

// row i of a packed symmetric matrix (zeros for lanes past nv and past nv in the row)
template <int NB>
DEV void load_row(const float* M, int i, int nv, float* A) {
#pragma unroll
  for (int j = 0; j < NB; j++) A[j] = 0.f;
  if (i < nv) {
    int at = tri(i, 0);
#pragma unroll
    for (int j = 0; j < NB; j++) {
      if (j < min_nv<NB>() || j < nv) A[j] = M[at];
      at += j < i ? 1 : j + 1;
    }
  }
}

// Newton's Hessian, summed up from a start (one row per lane) and the contacts' parts P J3 over
// their frames, and then solved with.  On the matrix cores for 32-lane teams (two worlds at once, a 32 x 32 block each) and
// 64-lane teams (two frames an instruction), by broadcast multiply-adds for 16 lanes.
// solve: this lane's entry of H^-1 b, and the rows A for times_inverse (scale: a factor of this
// lane).  ok: every pivot was positive.
template <int T, int NB>
struct SymAcc;
template <int NB>
struct SymAcc<16, NB> {
  float C[NB];
  DEV SymAcc(const float* R, int) {
#pragma unroll
    for (int j = 0; j < NB; j++) C[j] = R[j];
  }
  DEV void add(float p0, float j0, float p1, float j1) {
    dpp_axpy<16>(C, j0, p0);
    dpp_axpy<16>(C, j1, p1);
  }
  DEV void add1(float p, float j) { dpp_axpy<16>(C, j, p); }
  DEV float solve(int nv, int i, float b, float* A, float& scale, bool& ok) {
    const float x = sweep_inverse<16, NB>(C, scale, nv, i, b, ok);
#pragma unroll
    for (int j = 0; j < NB; j++) A[j] = C[j];
    return x;
  }
  DEV static float times_inverse(const float* A, float scale, float x) {
    return -scale * row_dot<NB>(A, rep_dof<16>(x));
  }
};
// The elimination on the matrix cores is the symmetric sweep with every swept row and column left
// unscaled: X_ij = -(H^-1)_ij p_i p_j off the diagonal, X_ii = 2 p_i - (H^-1)_ii p_i^2 at the
// end, p_i the pivots.  A pivot then is one symmetric rank-one update of the other rows,
// X -= v v^T / p (v: its row, 0 at the pivot), with no row or column to overwrite, and one
// matrix instruction whatever the size: 10 vector instructions and 64 clocks of the matrix core
// a pivot, against 28 (18 dofs) to 37 (28 dofs) vector instructions where each lane updated its
// row by broadcast multiply-adds.  FP32 matrix and vector instructions do not overlap here (with
// 65536 worlds their busy times add up to the whole), so 18 dofs gain in latency only: 64
// quadrupeds x 4 steps 148 -> 144 us, 8192 x 3 269 -> 254, 65536 x 1 410 -> 415; 8192 hands
// (22 dofs) x 4 730 -> 692, 2048 humanoids (27) x 2 160 -> 155.  The mass matrix, with one
// right-hand side, stays with gj_solve's half-length updates (64 quadrupeds 3.7 thousand clocks
// against 4.3).  Row and column 31, past every dof, carry the right-hand side.  Last dof first, as
// in gj_solve.
template <class Acc, int T, int NB>
struct SweepBase {
  template <int K>
  DEV static void pivot(Acc& S, int nv, int i, float& pd) {
    if (K < min_nv<NB>() || K < nv) {  // (nv is uniform)
      const float x = S.template row<K>();
      const float v = i == K ? 0.f : x;
      pd = i == K ? x : pd;
      const Pair w = swap16(x);
      const float p = row_bcast<(K & 15)>(K < 16 ? w.a : w.b);
      S.add1(-(v * __builtin_amdgcn_rcpf(p)), v);
    }
    if constexpr (K > 0) pivot<K - 1>(S, nv, i, pd);
  }
  DEV static float solve(Acc& S, const Team& t, int nv, int i, float b, float* A, float& scale,
                         bool& ok) {
    const float e31 = i == 31 ? 1.f : 0.f;
    // (an entry that is not finite, times e31's zeros, would spread from the right-hand side into
    // the matrix, whose pivots say whether it is positive definite: it stays out, and the
    // solution's entry is no number, which ends the solve at the descent test)
    const bool finite = fabsf(b) < INFINITY;
    S.add_rhs(finite ? b : 0.f, e31);
    float pd = 1.f;
    pivot<NB - 1>(S, nv, i, pd);
    ok = !team_any<T>(!(pd > 0.f), t.lane);
    scale = i < nv ? __builtin_amdgcn_rcpf(pd) : 0.f;  // (lane 31 holds the right-hand side)
    S.rows(A);
    const float x = scale * S.template row<31>();
    return finite ? x : NAN;
  }
};
template <int NB>
struct SymAcc<32, NB> {
  f32x32 C;  // block 0: the wavefront's first world, block 1 its second
  // block B's register v of lane l: its entry (8 (v / 4) + 4 (l / 32) + v % 4, l % 32); the
  // swaps give each half-wavefront its own block's two row groups, and back
  DEV SymAcc(const float* R, int) {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int r = 8 * (v >> 2) + (v & 3);
      const Pair h = r < NB ? swap32(R[r], r + 4 < NB ? R[r + 4] : 0.f) : Pair{0.f, 0.f};
      C[v] = h.a;
      C[16 + v] = h.b;
    }
  }
  DEV void add(float p0, float j0, float p1, float j1) {
    C = __builtin_amdgcn_mfma_f32_32x32x1f32(p0, j0, C, 0, 0, 0);
    C = __builtin_amdgcn_mfma_f32_32x32x1f32(p1, j1, C, 0, 0, 0);
  }
  DEV void add1(float p, float j) { C = __builtin_amdgcn_mfma_f32_32x32x1f32(p, j, C, 0, 0, 0); }
  DEV void add_rhs(float b, float e) { add(b, e, e, b); }
  template <int K>
  DEV float row() const {
    constexpr int v = 4 * (K >> 3) + (K & 3);
    const Pair h = swap32(C[v], C[16 + v]);
    return K & 4 ? h.b : h.a;
  }
  DEV void rows(float* A) const {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int r = 8 * (v >> 2) + (v & 3);
      if (r < NB) {
        const Pair h = swap32(C[v], C[16 + v]);
        A[r] = h.a;
        if (r + 4 < NB) A[r + 4] = h.b;
      }
    }
  }
};
template <int NB>
struct SymAcc<64, NB> {
  f32x16 C;
  bool up;
  // register v of lane l: entry (8 (v / 4) + 4 (l / 32) + v % 4, l % 32)
  DEV SymAcc(const float* R, int lane) : up(lane >= 32) {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int r = 8 * (v >> 2) + (v & 3);
      C[v] = r < NB ? (up ? (r + 4 < NB ? R[r + 4] : 0.f) : R[r]) : 0.f;
    }
  }
  DEV void add(float p0, float j0, float p1, float j1) {
    C = __builtin_amdgcn_mfma_f32_32x32x2f32(up ? p1 : p0, up ? j1 : j0, C, 0, 0, 0);
  }
  DEV void add1(float p, float j) {
    C = __builtin_amdgcn_mfma_f32_32x32x2f32(up ? 0.f : p, up ? 0.f : j, C, 0, 0, 0);
  }
  DEV void add_rhs(float b, float e) { add(b, e, e, b); }
  template <int K>
  DEV float row() const {
    constexpr int v = 4 * (K >> 3) + (K & 3);
    const Pair h = swap32(C[v], C[v]);
    return K & 4 ? h.b : h.a;
  }
  DEV void rows(float* A) const {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int r = 8 * (v >> 2) + (v & 3);
      if (r < NB) {
        const Pair h = swap32(C[v], C[v]);
        A[r] = h.a;
        if (r + 4 < NB) A[r + 4] = h.b;
      }
    }
  }
};
template <int T, int NB>
DEV float sym_solve(SymAcc<T, NB>& S, const Team& t, int nv, int i, float b, float* A,
                    float& scale, bool& ok) {
  if constexpr (T == 16) return S.solve(nv, i, b, A, scale, ok);
  else return SweepBase<SymAcc<T, NB>, T, NB>::solve(S, t, nv, i, b, A, scale, ok);
}
// this lane's entry of H^-1 x, from the rows that sym_solve left
template <int T, int NB>
DEV float times_inverse(const float* A, float scale, float x) {
  if constexpr (T == 16) return SymAcc<T, NB>::times_inverse(A, scale, x);
  // -scale (sum_j X_ij y_j - 2 p_i y_i), y = scale x
  else return -scale * row_dot<NB>(A, rep_dof<T>(scale * x), -2.f * x);
}

// x_i = (A^-1 rhs)_i for the mass matrix in o_M, plus h diag(dof_vgain) with hgain
template <int T, int NB>
DEV float smooth_solve_reg(const DevModel& m, float* W, const Team& t, float rhs, bool hgain) {
  const int i = T == 64 ? t.lane & 31 : t.lane, nv = m.nv;
  float A[NB];
  load_row<NB>(W + m.o_M, i, nv, A);
  if (hgain) {
    const float h = i < nv ? m.dt * m.dof_vgain[i] : 0.f;
#pragma unroll
    for (int j = 0; j < NB; j++) A[j] += j == i ? h : 0.f;
  }
  bool ok = true;
  return gj_solve<T, NB>(A, nv, i, rhs, ok);
}

// The constraint rows as the solvers see them.
template <int T, int NB>
struct RegRows {
  const DevModel& m;
  float* const W0;
  const int lane0;
  float* W;
  Team t;
  int i, nv, nrow, ncon, no, nl;  // dof of this lane; rows, contacts, others, active limits
  int ncu, nou;                   // the wavefront's largest contact and other-row counts
  bool dv;

  // a context of its own for the phase that follows (see opaque_zero)
  DEV void phase() {
    W = W0 + opaque_zero();
    t.lane = lane0 + opaque_zero();
  }
  DEV RegRows(const DevModel& m_, float* W_, const Team& t_)
      : m(m_), W0(W_), lane0(t_.lane), W(W_), t(t_) {
    const int* scal = (const int*)(W + m.o_scal);
    i = T == 64 ? t.lane & 31 : t.lane;
    nv = m.nv;
    dv = i < nv;
    nrow = scal[SC_NROW];
    ncon = scal[SC_NCON];
    no = nrow - 4 * ncon;
    nl = no - m.nfric - m.neqrow;
    ncu = wave_max<T>(ncon);
    nou = wave_max<T>(no);
  }
  // J row f . x (all lanes take part; finite rows only); FINE: summed in FP64
  template <bool FINE>
  DEV float j_dot(int f, const Pair& x) const {
    const float* Jr = W + m.o_J + f * nv;
    float J[NB];
#pragma unroll
    for (int j = 0; j < NB; j++) {
      J[j] = 0.f;
      if (j < min_nv<NB>() || j < nv) J[j] = Jr[j];
    }
    if constexpr (FINE) {
      double acc = 0.0;
      fine_dot<0>(acc, J, x);
      return (float)acc;
    }
    return row_dot<NB>(J, x);
  }
  template <int K>
  DEV void fine_dot(double& acc, const float* J, const Pair& x) const {
    acc += (double)J[K] * (double)row_bcast<(K & 15)>(K < 16 ? x.a : x.b);
    if constexpr (K + 1 < NB) fine_dot<K + 1>(acc, J, x);
  }
  DEV float mu(int c) const { return W[m.o_con + kConRec * c + 13]; }
  // f(r, v) for every row r of the world that this lane holds, v = J_r x (x: this lane's
  // entry of a dof vector).  A contact's quad: lanes 0, 1, 2 form J_n x, J_t1 x, J_t2 x.
  template <bool FINE = false, class F>
  DEV void times(float x, F f) const {
    const Pair xr = rep_dof<T>(x);
    const int q = t.lane & 3;
    for (int cb = 0; cb < ncu; cb += T / 4) {
      const int c = cb + (t.lane >> 2);
      const bool act = c < ncon;
      const float v = j_dot<FINE>(act ? 3 * c + min(q, 2) : 0, xr);
      const float vn = quad_perm<0x00>(v), vt = quad_perm<0xA5>(v);
      const float mc = act ? mu(c) : 0.f;
      if (act) f(4 * c + q, vn + ((q & 1) ? -mc : mc) * vt);
    }
    for (int kb = 0; kb < nou; kb += T) {
      const int k = kb + t.lane;
      const bool act = k < no;
      int dof = 0;
      float sg = 1.f;
      bool unit = true;
      if (act && k < nl) limit_sign(k, dof, sg);
      else if (act && k < nl + m.nfric) dof = m.fric_dadr[k - nl];
      else unit = !act;
      float v = sg * from_dof(x, dof);
      if (m.neqrow > 0) {
        const float vd = j_dot<FINE>(act ? 3 * ncon + k : 0, xr);
        v = unit ? v : vd;
      }
      if (act) f(4 * ncon + k, v);
    }
  }
  DEV float from_dof(float x, int dof) const {
    const int base = (int)(threadIdx.x & 63) - t.lane;
    return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (base + dof), __float_as_int(x)));
  }
  DEV void limit_sign(int k, int& dof, float& sg) const {
    const int code = ((const int*)(W + m.o_lim))[k];
    dof = m.lim_dadr[code & 0xffff];
    sg = (code >> 16) ? -1.f : 1.f;
  }
  // the words of Newton's vectors in LDS are free here: per-dof slots of the unit rows
  DEV float* unit_slots(int which) const { return W + m.o_Mr + which * nv; }
  DEV void clear_units() const {
    if (nou > 0)
      for (int k = t.lane; k < 4 * nv; k += T) unit_slots(0)[k] = 0.f;
  }
  // scatter y(r) (times the row's sign when signed) of the unit rows into two slots per dof:
  // a dof has at most one active limit and one friction-loss row
  template <class Y>
  DEV void put_units(int slot, bool sign, Y y) const {
    for (int kb = 0; kb < nou; kb += T) {
      const int k = kb + t.lane;
      if (k < nl) {
        int dof;
        float sg;
        limit_sign(k, dof, sg);
        unit_slots(slot)[dof] = sign ? sg * y(4 * ncon + k) : y(4 * ncon + k);
      } else if (k < nl + m.nfric) {
        unit_slots(slot + 1)[m.fric_dadr[k - nl]] = y(4 * ncon + k);
      }
    }
  }
  DEV float get_units(int slot) const {
    return dv && nou > 0 ? unit_slots(slot)[i] + unit_slots(slot + 1)[i] : 0.f;
  }
  // entry i of frame rows 3c, 3c + 1, 3c + 2 (0 past this world's contacts and dofs)
  DEV void frame_col(int c, float& n, float& a, float& b) const {
    const float* Jc = W + m.o_J + 3 * c * nv + i;
    n = a = b = 0.f;
    if (dv && c < ncon) {
      n = Jc[0];
      a = Jc[nv];
      b = Jc[2 * nv];
    }
  }
  // init_i + sum_r y(r) J_ri, y a functor over this world's rows
  template <class Y>
  DEV float t_times(Y y, float init) const {
    float* fy = W + m.o_fw;
    const int q = t.lane & 3;
    for (int cb = 0; cb < ncu; cb += T / 4) {
      const int c = cb + (t.lane >> 2);
      const bool act = c < ncon;
      const float yr = act ? y(4 * c + q) : 0.f, mc = act ? mu(c) : 0.f;
      const float yx = quad_perm<kXor1>(yr);
      const float sm = yr + yx, df = yr - yx;  // lanes 0 and 2: the pairs' sums, differences
      const float all = sm + quad_perm<kXor2>(sm);
      if (c < ncu && !(q & 1)) {
        if (q == 0) fy[3 * c] = all;
        fy[3 * c + 1 + (q >> 1)] = mc * df;
      }
    }
    put_units(0, true, y);
    t.sync();
    float v = init;
    for (int c = 0; c < ncu; c++) {
      float n, a, b;
      frame_col(c, n, a, b);
      v += fy[3 * c] * n;
      v += fy[3 * c + 1] * a;
      v += fy[3 * c + 2] * b;
    }
    v += get_units(0);
    const int e0 = 3 * ncon + nl + m.nfric;  // the equality rows, always present
    for (int k = 0; k < m.neqrow; k++)
      if (dv && nrow > 0) v += y(4 * ncon + nl + m.nfric + k) * W[m.o_J + (e0 + k) * nv + i];
    t.sync();
    return v;
  }
  // Mrow + sum_r w(r) J_ri J_r. (row i of the Hessian), w the rows' weights
  template <class Wt>
  DEV SymAcc<T, NB> hessian(const float* Mrow, Wt w) const {
    float* cf = W + m.o_fw;
    const int q = t.lane & 3;
    for (int cb = 0; cb < ncu; cb += T / 4) {
      const int c = cb + (t.lane >> 2);
      const bool act = c < ncon;
      const float wr = act ? w(4 * c + q) : 0.f, mc = act ? mu(c) : 0.f;
      const float wx = quad_perm<kXor1>(wr);
      const float sm = wr + wx, df = wr - wx;
      const float all = sm + quad_perm<kXor2>(sm);
      if (c < ncu && !(q & 1)) {
        if (q == 0) cf[5 * c] = all;
        cf[5 * c + 1 + q] = mc * df;
        cf[5 * c + 2 + q] = mc * mc * sm;
      }
    }
    put_units(2, false, w);
    t.sync();
    // a contact adds P J3 over its frames, P = J3^T C: rows P_f of this lane's dof
    const int e0 = 3 * ncon + nl + m.nfric;
    float A[NB];
    const float du = nou > 0 ? get_units(2) : 0.f;
#pragma unroll
    for (int j = 0; j < NB; j++) A[j] = Mrow[j] + (j == i ? du : 0.f);
    SymAcc<T, NB> acc(A, t.lane);
    for (int c = 0; c < ncu; c++) {
      float n, a, b;
      frame_col(c, n, a, b);
      const float* k = cf + 5 * c;
      const float pn = k[0] * n + k[1] * a + k[3] * b;
      const float pa = k[1] * n + k[2] * a, pb = k[3] * n + k[4] * b;
      acc.add(pn, n, pa, a);
      acc.add1(pb, b);
    }
    for (int k = 0; k < m.neqrow; k++) {
      const float j = dv && nrow > 0 ? W[m.o_J + (e0 + k) * nv + i] : 0.f;
      const float wk = nrow > 0 ? w(4 * ncon + nl + m.nfric + k) : 0.f;
      acc.add1(wk * j, j);
    }
    t.sync();
    return acc;
  }
};

// sum over the 16 rows held by one replicated 16-lane row (up to n of them, n uniform) of the
// line search's slope terms
template <int B = 0>
DEV float slope_rows(float dp, float e, float s, float ds, float br, int n) {
  if (n > B) {
    dp = dpp_slope4<B>(dp, e, s, ds, br);
    if constexpr (B < 12) return slope_rows<B + 4>(dp, e, s, ds, br, n);
  }
  return dp;
}
// the same for rows with a force bound F (row_slope): one row per step
template <int K = 0>
DEV float slope_rows_fr(float dp, float e, float s, float D, float F, float br, int n) {
  if (n > K) {
    const float sq = row_bcast<K>(s);
    dp += sq * row_slope(row_bcast<K>(D), row_bcast<K>(F), row_bcast<K>(e) + br * sq);
    if constexpr (K < 15) return slope_rows_fr<K + 1>(dp, e, s, D, F, br, n);
  }
  return dp;
}
// a row vector's 16-lane rows, each replicated over the team
template <int T>
struct RowRep {
  float r[T / 16];
  DEV explicit RowRep(float x) {
    if constexpr (T == 16) {
      r[0] = x;
    } else if constexpr (T == 32) {
      const Pair p = swap16(x);
      r[0] = p.a;
      r[1] = p.b;
    } else {
      const Pair h = swap32(x, x), lo = swap16(h.a), hi = swap16(h.b);
      r[0] = lo.a;
      r[1] = lo.b;
      r[2] = hi.a;
      r[3] = hi.b;
    }
  }
};

// newton_impl's solve (see there for the steps and the stopping rules), rows in chunks of T
template <int T, int NB, bool FR>
DEV void newton_chunks(const DevModel& m, int& status, int iters, RegRows<T, NB>& R, int nru) {
  const Team& t = R.t;
  // the row arrays (through the phase's base, so that no address is held across phases)
  auto e = [&](int r) -> float& { return R.W[m.o_e + r]; };   // J a - aref
  auto s = [&](int r) -> float& { return R.W[m.o_s + r]; };   // J delta
  auto D = [&](int r) { return R.W[m.o_D + r]; };
  auto fl = [&](int r) { return FR ? R.W[m.o_fl + r] : 0.f; };
  const int nrow = R.nrow, i = R.i, nv = m.nv;
  const bool dv = R.dv;
  const float a0 = dv ? R.W[m.o_a0 + i] : 0.f;
  bool done = nrow == 0;
  float a = dv ? R.W[m.o_qacc + i] : 0.f;
  float Mrow[NB];
  load_row<NB>(R.W + m.o_M, i, nv, Mrow);
  R.clear_units();  // (the poses and motion subspaces there are dead from here on)
  // constraint_rows leaves aref's distance term: add -B (J qvel)
  R.times(dv ? R.W[m.o_qvel + i] : 0.f, [&](int r, float v) { R.W[m.o_aref + r] -= m.B * v; });
  t.sync();
  // ---- start point: cost of the warm start vs cost of a0
  const float Mw = row_dot<NB>(Mrow, rep_dof<T>(a - a0));
  float cw = 0.f, c0 = 0.f;
  auto cost = [&](int r, float v) {
    return FR ? row_cost(D(r), fl(r), v) : (v < 0.f ? 0.5f * D(r) * v * v : 0.f);
  };
  R.times(a, [&](int r, float v) { cw += cost(r, v - R.W[m.o_aref + r]); });
  R.times(a0, [&](int r, float v) { c0 += cost(r, v - R.W[m.o_aref + r]); });
  cw = t.sum(cw) + dof_sum<T>(t, 0.5f * (a - a0) * Mw);
  c0 = t.sum(c0);
  if (!(cw <= c0) || done) a = a0;
  // the residuals are small differences of large terms (a stiff contact's D e is its force)
  // and later steps only add to them: their start is summed in FP64
  R.template times<true>(a, [&](int r, float v) { e(r) = v - R.W[m.o_aref + r]; });
  t.sync();
  // the smooth part of the gradient, M (a - a0), as M a - frc: a0's own rounding, which M
  // multiplies and which is large where a0 is (a leg pressed into the ground), stays out of it
  float Mr = row_dot<NB>(Mrow, rep_dof<T>(a), dv ? -R.W[m.o_frc + i] : 0.f);
  t.sync();
  auto quad = [&](int r) { return FR ? row_quad(D(r), fl(r), e(r)) : e(r) < 0.f; };
  auto rep = [&](float x) { return rep_dof<T>(x); };
  float A[NB], sc = 1.f;  // the Hessian's inverse (times_inverse)
#pragma unroll
  for (int j = 0; j < NB; j++) A[j] = 0.f;
  bool kept = false;      // A holds the inverse at the current pieces
  for (int it = 0; it < iters; it++) {
    R.phase();
    const float g = R.t_times([&](int r) {
      const float er = e(r);
      return FR ? row_slope(D(r), fl(r), er) : (er < 0.f ? D(r) * er : 0.f);
    }, Mr);
    if (!__ballot(!done)) break;
    // ---- delta = -H^-1 g.  With no piece changed by the last step the inverse is that of the
    // last iteration (and comes out the same if the wavefront's other world needs a new one);
    // then the direction is a product with it, else it comes out of the elimination.
    float de = 0.f;
    bool ok = true;
    if (__ballot(!done && !kept)) {
      R.phase();
      SymAcc<T, NB> S = R.hessian(Mrow, [&](int r) { return quad(r) ? D(r) : 0.f; });
      de = sym_solve<T, NB>(S, t, nv, i, -g, A, sc, ok);
    }
    float d = de;
    if (__ballot(kept)) d = kept ? -times_inverse<T, NB>(A, sc, g) : de;
    if (!kept && !done && !ok) {
      status |= 4;
      done = true;
    }
    // ---- one step of iterative refinement, H applied unassembled
    R.phase();
    R.times(d, [&](int r, float v) { s(r) = quad(r) ? D(r) * v : 0.f; });
    const float res = R.t_times([&](int r) { return s(r); }, row_dot<NB>(Mrow, rep(d), g));
    const float corr = times_inverse<T, NB>(A, sc, res);
    d -= corr;
    const float cm = dof_max<T>(t, fabsf(corr));
    // ---- line search quantities
    R.phase();
    const float Md = row_dot<NB>(Mrow, rep(d));
    R.times(d, [&](int r, float v) { s(r) = v; });
    const float gd = dof_sum<T>(t, g * d), dMd = dof_sum<T>(t, d * Md),
                dMr = dof_sum<T>(t, d * Mr);
    t.sync();
    done = done || !(gd < 0.f);
    // ---- phi' at every positive breakpoint (one candidate a lane)
    float lo = 0.f, hi = INFINITY;
    const int nbp = FR ? nrow + m.nfric : nrow;
    const int nbu = FR ? nru + m.nfric : nru;
    const int nfr0 = nrow - m.nfric - m.neqrow;  // first friction-loss row
    for (int cb = 0; cb < nbu; cb += T) {
      const int c = cb + t.lane;
      float br = 0.f;
      if (c < nbp) {
        const int r = c < nrow ? c : nfr0 + (c - nrow);
        const float sr = s(r);
        float at = 0.f;
        bool use = sr != 0.f;
        if (FR && fl(r) > 0.f) {
          use = use && fl(r) != INFINITY;
          at = (c < nrow ? fl(r) : -fl(r)) / D(r);
        }
        if (use) br = (at - e(r)) / sr;
      }
      float dp = dMr + br * dMd;
      for (int rb = 0; rb < nru; rb += T) {
        const int r = rb + t.lane;
        const bool in = r < nrow;
        const float er = in ? e(r) : 0.f, sr = in ? s(r) : 0.f, Dr = in ? D(r) : 0.f;
        const RowRep<T> re(er), rs(sr), rd(FR ? Dr : Dr * sr);
        const RowRep<T> rf(FR && in ? fl(r) : 0.f);
#pragma unroll
        for (int h = 0; h < T / 16; h++) {
          const int n = nru - rb - 16 * h;
          if constexpr (FR) dp = slope_rows_fr<>(dp, re.r[h], rs.r[h], rd.r[h], rf.r[h], br, n);
          else dp = slope_rows<>(dp, re.r[h], rs.r[h], rd.r[h], br, n);
        }
      }
      if (br > 0.f) {
        if (dp <= 0.f) lo = fmaxf(lo, br);
        else hi = fminf(hi, br);
      }
    }
    lo = t.max(lo);
    hi = t.min(hi);
    R.phase();
    const float probe = (hi < INFINITY) ? 0.5f * (lo + hi) : lo + 1.f;
    float Ac = 0.f, Bc = 0.f;
    for (int r = t.lane; r < nrow; r += T) {
      const float sr = s(r), er = e(r), Dr = D(r), ep = er + probe * sr;
      if (FR ? row_quad(Dr, fl(r), ep) : ep < 0.f) {
        Ac += Dr * sr * er;
        Bc += Dr * sr * sr;
      } else if (FR) {
        Ac += sr * row_slope(Dr, fl(r), ep);
      }
    }
    Ac = t.sum(Ac) + dMr;
    Bc = t.sum(Bc) + dMd;
    float al = -Ac / Bc;
    al = fminf(fmaxf(al, lo), hi);
    // ---- update
    bool moved = false;
    if (!done) {
      a += al * d;
      Mr += al * Md;
      for (int r = t.lane; r < nrow; r += T) {
        const float e0 = e(r), e1 = e0 + al * s(r);
        moved = moved || (FR ? (row_piece(D(r), fl(r), e0) != row_piece(D(r), fl(r), e1))
                             : ((e0 < 0.f) != (e1 < 0.f)));
        e(r) = e1;
      }
    }
    moved = team_any<T>(moved, R.lane0);
    const float am = dof_max<T>(t, fmaxf(1.f, fabsf(a)));
    t.sync();
    done = done || (!moved && cm <= kNewtonExitTol * am);
    kept = !moved;
  }
  if (dv) R.W[m.o_qacc + i] = a;
  t.sync();
}

// The same solve for at most T rows: row r's state (residual, curvature, Jacobian row) is in
// lane r's registers too, so that an iteration reads LDS only for the frame rows' columns.
// Lane r < 4 ncon holds edge r (its quad's lanes 0, 1, 2 the frame rows), the others a limit,
// friction-loss or equality row.  Against the rows in LDS (newton_chunks, still the solve for
// more rows than lanes): 64 quadrupeds x 4 steps 204 -> 173 us, 8192 x 3 steps 327 -> 288 us,
// 2048 humanoids x 2 steps 198 -> 182 us, 8192 hands x 4 steps 945 -> 847 us; what that bought is
// LDS round trips, on which these short phases wait.
template <int T, int NB, bool FR>
struct LaneRows {
  RegRows<T, NB>& R;
  const DevModel& m;
  float J[NB];
  float e, D, F, smu, zc;  // F: force bound (FR); smu: +-mu of an edge; zc: see fold
  bool con, act, eq;       // a contact's edge; a row of this world; an equality row
  int dof;                 // dof and sign of a unit row, else -1
  float sg;

  DEV LaneRows(RegRows<T, NB>& R_, const DevModel& m_) : R(R_), m(m_) {
    const int r = R.t.lane, c = r >> 2, q = r & 3, k = r - 4 * R.ncon;
    con = r < 4 * R.ncon;
    act = r < R.nrow;
    const int f = con ? 3 * c + min(q, 2) : (act ? r - R.ncon : 0);  // (any words past them)
    const float* Jr = R.W + m.o_J + f * R.nv;
#pragma unroll
    for (int j = 0; j < NB; j++) {
      J[j] = 0.f;
      if (j < min_nv<NB>() || j < R.nv) J[j] = Jr[j];
    }
    const float mc = con ? R.mu(c) : 0.f;
    smu = (q & 1) ? -mc : mc;
    zc = q == 1 ? -mc : (q == 2 ? mc : 0.f);
    D = act ? R.W[m.o_D + r] : 0.f;
    F = FR && act ? R.W[m.o_fl + r] : 0.f;
    dof = -1;
    sg = 1.f;
    eq = act && k >= R.nl + m.nfric;
    if (act && k >= 0 && k < R.nl) R.limit_sign(k, dof, sg);
    else if (act && k >= R.nl && !eq) dof = m.fric_dadr[k - R.nl];
  }
  // J_r x (0 past the world's rows)
  template <bool FINE = false>
  DEV float times(float x) const {
    const Pair xr = rep_dof<T>(x);
    float v;
    if constexpr (FINE) {
      double acc = 0.0;
      R.template fine_dot<0>(acc, J, xr);
      v = (float)acc;
    } else {
      v = row_dot<NB>(J, xr);
    }
    const float vn = quad_perm<0x00>(v), vt = quad_perm<0xA5>(v);
    return con ? vn + smu * vt : (act ? v : 0.f);
  }
  // a row vector folded onto the contacts' frames: lanes 0, 1, 2 of a quad hold sum y,
  // mu (y0 - y1), mu (y2 - y3)
  DEV float fold(float y) const {
    const float yx = quad_perm<kXor1>(y), sm = y + yx;
    const float all = sm + quad_perm<kXor2>(sm);
    return (R.t.lane & 3) == 0 ? all : zc * (y - yx);
  }
  template <int C>
  DEV float add_contacts(float v, const RowRep<T>& z) const {
    if (C < R.ncu) {
      float n, a, b;
      R.frame_col(C, n, a, b);
      v = dpp_quad3<4 * (C & 3)>(v, z.r[C >> 2], n, a, b);
      if constexpr (C + 1 < T / 4) return add_contacts<C + 1>(v, z);
    }
    return v;
  }
  // init_i + sum_r y_r J_ri on dof lane i
  DEV float t_times(float y, float init) const {
    float v = init;
    if (R.nou > 0) put(0, sg * y);
    if (R.ncu > 0) v = add_contacts<0>(v, RowRep<T>(fold(y)));
    if (R.nou > 0) {
      R.t.sync();
      v += R.get_units(0);
      v += equalities(y);
      R.t.sync();
    }
    return v;
  }
  DEV void put(int slot, float y) const {  // unit rows: slot for limits, the next for friction
    if (dof >= 0) R.unit_slots(slot + (R.t.lane - 4 * R.ncon >= R.nl ? 1 : 0))[dof] = y;
  }
  DEV float equalities(float y) const {
    float v = 0.f;
    const int base = (int)(threadIdx.x & 63) - R.t.lane;
    for (int k = 0; k < m.neqrow; k++) {
      const int r = max(R.nrow - m.neqrow + k, 0);
      const float yk = __int_as_float(
          __builtin_amdgcn_ds_bpermute(4 * (base + r), __float_as_int(y)));
      if (R.dv && R.nrow > 0) v += yk * R.W[m.o_J + (r - R.ncon) * R.nv + R.i];
    }
    return v;
  }
  template <int C, class Acc>
  DEV void hess_contacts(const RowRep<T>& all, const RowRep<T>& d, const RowRep<T>& s,
                         Acc& acc) const {
    if (C < R.ncu) {
      float n, a, b, pn, pa, pb;
      R.frame_col(C, n, a, b);
      dpp_frame<4 * (C & 3)>(all.r[C >> 2], d.r[C >> 2], s.r[C >> 2], n, a, b, pn, pa, pb);
      acc.add(pn, n, pa, a);
      acc.add1(pb, b);
      if constexpr (C + 1 < T / 4) hess_contacts<C + 1>(all, d, s, acc);
    }
  }
  // Mrow + sum_r w_r J_ri J_r.
  DEV SymAcc<T, NB> hessian(const float* Mrow, float w) const {
    float A[NB];
#pragma unroll
    for (int j = 0; j < NB; j++) A[j] = Mrow[j];
    if (R.nou > 0) {
      put(2, w);
      R.t.sync();
      const float du = R.get_units(2);
#pragma unroll
      for (int j = 0; j < NB; j++) A[j] += j == R.i ? du : 0.f;
      R.t.sync();
    }
    SymAcc<T, NB> acc(A, R.t.lane);
    if (R.ncu > 0) {
      const float wc = con ? w : 0.f, wx = quad_perm<kXor1>(wc), sm = wc + wx;
      const float mc = fabsf(smu);
      const RowRep<T> all(sm + quad_perm<kXor2>(sm)), d(mc * (wc - wx)), s(mc * mc * sm);
      hess_contacts<0>(all, d, s, acc);
    }
    if (R.nou > 0) {
      const int base = (int)(threadIdx.x & 63) - R.t.lane;
      for (int k = 0; k < m.neqrow; k++) {
        const int r = max(R.nrow - m.neqrow + k, 0);
        const float wk = __int_as_float(
            __builtin_amdgcn_ds_bpermute(4 * (base + r), __float_as_int(w)));
        const float j = R.dv && R.nrow > 0 ? R.W[m.o_J + (r - R.ncon) * R.nv + R.i] : 0.f;
        acc.add1(wk * j, j);
      }
    }
    return acc;
  }
};

// dp + sum over rows of ds min(0, e + br s), n rows (uniform); the T-lane vectors replicated
template <int T>
DEV float slope_sum(float dp, const RowRep<T>& e, const RowRep<T>& s, const RowRep<T>& ds, float br,
                    int n) {
#pragma unroll
  for (int h = 0; h < T / 16; h++)
    if (n > 16 * h) dp = slope_rows<>(dp, e.r[h], s.r[h], ds.r[h], br, n - 16 * h);
  return dp;
}

// dp + sum over rows of s clamp(D (e + br s), lo, hi), likewise
template <int B = 0>
DEV float clamp_rows(float dp, float e, float s, float D, float lo, float hi, float br, int n) {
  if (n > B) {
    dp = dpp_clamp4<B>(dp, e, s, D, lo, hi, br);
    if constexpr (B < 12) return clamp_rows<B + 4>(dp, e, s, D, lo, hi, br, n);
  }
  return dp;
}
template <int T>
DEV float clamp_sum(float dp, const RowRep<T>& e, const RowRep<T>& s, const RowRep<T>& D,
                    const RowRep<T>& lo, const RowRep<T>& hi, float br, int n) {
#pragma unroll
  for (int h = 0; h < T / 16; h++)
    if (n > 16 * h)
      dp = clamp_rows<>(dp, e.r[h], s.r[h], D.r[h], lo.r[h], hi.r[h], br, n - 16 * h);
  return dp;
}

template <int T, int NB, bool FR>
DEV void newton_rows(const DevModel& m, int& status, int iters, RegRows<T, NB>& R, int nru) {
  const Team& t = R.t;
  const int nrow = R.nrow, i = R.i, nv = m.nv, lane = R.lane0;
  const bool dv = R.dv;
  const float a0 = dv ? R.W[m.o_a0 + i] : 0.f;
  bool done = nrow == 0;
  float a = dv ? R.W[m.o_qacc + i] : 0.f;
  LaneRows<T, NB, FR> L(R, m);
  // constraint_rows leaves the distance term; the rows are here to add -B (J qvel)
  const float aref = (lane < nrow ? R.W[m.o_aref + lane] : 0.f) -
                     m.B * L.times(dv ? R.W[m.o_qvel + i] : 0.f);
  if (lane < nrow) R.W[m.o_aref + lane] = aref;
  float Mrow[NB];
  load_row<NB>(R.W + m.o_M, i, nv, Mrow);
  R.clear_units();
  auto rep = [&](float x) { return rep_dof<T>(x); };
  auto cost = [&](float v) {  // (rows past the world's have D = 0)
    return FR ? (L.D > 0.f ? row_cost(L.D, L.F, v) : 0.f) : (v < 0.f ? 0.5f * L.D * v * v : 0.f);
  };
  auto quad = [&](float v) { return FR ? row_quad(L.D, L.F, v) : v < 0.f; };
  auto slope = [&](float v) {
    return FR ? row_slope(L.D, L.F, v) : (v < 0.f ? L.D * v : 0.f);
  };
  // ---- start point
  {
    const float Mw = row_dot<NB>(Mrow, rep(a - a0));
    const Pair c = sum2<T>(cost(L.times(a) - aref), cost(L.times(a0) - aref));
    const float cw = c.a + dof_sum<T>(t, 0.5f * (a - a0) * Mw);
    if (!(cw <= c.b) || done) a = a0;
  }
  L.e = L.template times<true>(a) - aref;
  float Mr = row_dot<NB>(Mrow, rep(a), dv ? -R.W[m.o_frc + i] : 0.f);
  t.sync();
  float A[NB], sc = 1.f;  // the Hessian's inverse (times_inverse)
#pragma unroll
  for (int j = 0; j < NB; j++) A[j] = 0.f;
  bool kept = false;
  for (int it = 0; it < iters; it++) {
    R.phase();
    const float g = L.t_times(slope(L.e), Mr);
    if (!__ballot(!done)) break;
    float de = 0.f;
    bool ok = true;
    const bool on = quad(L.e);  // on the quadratic piece
    if (__ballot(!done && !kept)) {
      SymAcc<T, NB> S = L.hessian(Mrow, on ? L.D : 0.f);
      de = sym_solve<T, NB>(S, t, nv, i, -g, A, sc, ok);
    }
    float d = de;
    if (__ballot(kept)) d = kept ? -times_inverse<T, NB>(A, sc, g) : de;
    if (!kept && !done && !ok) {
      status |= 4;
      done = true;
    }
    // ---- refinement
    R.phase();
    const float sd = L.times(d);
    const float res = L.t_times(on ? L.D * sd : 0.f, row_dot<NB>(Mrow, rep(d), g));
    const float corr = times_inverse<T, NB>(A, sc, res);
    d -= corr;
    // ---- line search
    const float s = L.times(d);
    const float Md = row_dot<NB>(Mrow, rep(d));
    const float gd = dof_sum<T>(t, g * d);
    const Pair dM = dof_sum2<T>(d * Md, d * Mr);
    const float dMd = dM.a, dMr = dM.b;
    done = done || !(gd < 0.f);
    float lo = 0.f, hi = INFINITY;
    {
      const RowRep<T> rs(s);
      float br = 0.f, br2 = 0.f;
      if (!FR) {
        if (s != 0.f) br = -L.e / s;
        const float dp = slope_sum<T>(dMr + br * dMd, RowRep<T>(L.e), rs, RowRep<T>(L.D * s), br, nru);
        if (br > 0.f) {
          if (dp <= 0.f) lo = br;
          else hi = br;
        }
      } else {
        // every row's slope is clamp(D v, lo, hi): (-inf, 0) one-sided, (-F, F) friction loss,
        // (-inf, inf) an equality row.  Clamped as it stands: written as one-sided terms shifted
        // by +-F / D with F s summed apart, the terms cancelled and lost digits as F outgrew the
        // forces (quadrupeds with F = 1e7: accelerations off by up to 7 %)
        const bool two = L.F > 0.f && L.F < INFINITY;
        const float sh = two ? L.F / L.D : 0.f;
        if (s != 0.f && !L.eq) {
          br = (sh - L.e) / s;
          if (two) br2 = (-sh - L.e) / s;
        }
        const RowRep<T> re(L.e), rD(L.D), rlo(L.F > 0.f ? -L.F : -INFINITY), rhi(L.F);
        auto at = [&](float b) {
          return clamp_sum<T>(dMr + b * dMd, re, rs, rD, rlo, rhi, b, nru);
        };
        const float dp = at(br);
        if (br > 0.f) {
          if (dp <= 0.f) lo = br;
          else hi = br;
        }
        if (m.nfric > 0) {
          const float dp2 = at(br2);
          if (br2 > 0.f) {
            if (dp2 <= 0.f) lo = fmaxf(lo, br2);
            else hi = fminf(hi, br2);
          }
        }
      }
    }
    const Pair lh = max2<T>(lo, -hi);
    lo = lh.a;
    hi = -lh.b;
    const float probe = (hi < INFINITY) ? 0.5f * (lo + hi) : lo + 1.f;
    const float ep = L.e + probe * s;
    const bool pq = quad(ep);
    float Ac = pq ? L.D * s * L.e : 0.f, Bc = pq ? L.D * s * s : 0.f;
    if (FR && !pq) Ac = s * row_slope(L.D, L.F, ep);
    const Pair AB = sum2<T>(Ac, Bc);
    Ac = AB.a + dMr;
    Bc = AB.b + dMd;
    float al = -Ac / Bc;
    al = fminf(fmaxf(al, lo), hi);
    // ---- update
    bool moved = false;
    if (!done) {
      a += al * d;
      Mr += al * Md;
      const float e1 = L.e + al * s;
      moved = FR ? row_piece(L.D, L.F, L.e) != row_piece(L.D, L.F, e1)
                 : (L.e < 0.f) != (e1 < 0.f);
      L.e = e1;
    }
    moved = team_any<T>(moved && lane < nrow, lane);
    const Pair ca = dof_max2<T>(fabsf(corr), fmaxf(1.f, fabsf(a)));
    done = done || (!moved && ca.a <= kNewtonExitTol * ca.b);
    kept = !moved;
  }
  if (lane < nrow) R.W[m.o_e + lane] = L.e;
  if (dv) R.W[m.o_qacc + i] = a;
  t.sync();
}

template <int T, int NB, bool FR>
DEV void newton_reg(const DevModel& m, float* W, const Team& t, int& status, int iters) {
  RegRows<T, NB> R(m, W, t);
  const int nru = wave_max<T>(R.nrow);
  if (nru == 0) {
    if (R.dv) W[m.o_qacc + R.i] = W[m.o_a0 + R.i];
    t.sync();
  } else if (nru <= T) {
    newton_rows<T, NB, FR>(m, status, iters, R, nru);
  } else {
    newton_chunks<T, NB, FR>(m, status, iters, R, nru);
  }
}

// implicit_damping with the registers' elimination
template <int T, int NB>
DEV void implicit_damping_reg(const DevModel& m, float* W, const Team& t) {
  const RegRows<T, NB> R(m, W, t);
  const float* D = W + m.o_D;
  const float* e = W + m.o_e;
  const float* fl = W + m.o_fl;
  const bool fr = has_bounds(m), dv = R.dv;
  const int i = R.i;
  float rhs = dv ? W[m.o_frc + i] : 0.f;
  if (m.implicit == 2 && dv) rhs -= m.dof_hkp[i] * W[m.o_qvel + i];
  R.clear_units();
  t.sync();
  rhs = R.t_times([&](int r) {
    return -(fr ? row_slope(D[r], fl[r], e[r]) : fminf(D[r] * e[r], 0.f));
  }, rhs);
  const float x = smooth_solve_reg<T, NB>(m, W, t, rhs, true);
  if (dv) W[m.o_frc + i] = x;
  t.sync();
}

}  // namespace mjh
