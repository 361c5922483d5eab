// Cross-lane building blocks of the register-resident linear algebra.
//
// A world's dof vector lives one entry per lane: entry i on lane i of its team (a 64-lane
// team holds it twice, on lanes i and i + 32), and a symmetric matrix one row per lane,
// A[j] being entry (i, j).  Products and eliminations need entry k of such a vector on
// every lane.  A DPP operand can broadcast lane k of each 16-lane row to that row at no
// cost (row_newbcast), fused into the multiply-add itself, once the vector's 16-lane rows
// are replicated to every row of the team: one permlane swap.  A broadcast multiply-add
// then takes one instruction and no LDS, against a readlane per team, a select and the
// FMA, or an LDS write, a wait and a read.
#pragma once
#include <hip/hip_runtime.h>

namespace mjh {

typedef float f32x32 __attribute__((ext_vector_type(32)));

// The compiler does not fuse a DPP move into a multiply-add, so the blocks are written out.
// Each starts with the two wait states a DPP read needs after its source was written; a block
// whose result may be read next by a DPP or matrix instruction also ends with them, because
// the compiler's hazard checks do not look into the blocks.
#define MJH_AX(d) "v_fmac_f32_dpp %" #d ", %[c], %[b] row_newbcast:" #d " row_mask:0xf bank_mask:0xf\n"
#define MJH_AX4 MJH_AX(0) MJH_AX(1) MJH_AX(2) MJH_AX(3)
#define MJH_AX8 MJH_AX4 MJH_AX(4) MJH_AX(5) MJH_AX(6) MJH_AX(7)
#define MJH_AX12 MJH_AX8 MJH_AX(8) MJH_AX(9) MJH_AX(10) MJH_AX(11)
#define MJH_AX16 MJH_AX12 MJH_AX(12) MJH_AX(13) MJH_AX(14) MJH_AX(15)
#define MJH_O4 "+v"(A[0]), "+v"(A[1]), "+v"(A[2]), "+v"(A[3])
#define MJH_O8 MJH_O4, "+v"(A[4]), "+v"(A[5]), "+v"(A[6]), "+v"(A[7])
#define MJH_O12 MJH_O8, "+v"(A[8]), "+v"(A[9]), "+v"(A[10]), "+v"(A[11])
#define MJH_O16 MJH_O12, "+v"(A[12]), "+v"(A[13]), "+v"(A[14]), "+v"(A[15])
// A[k] += (lane k of c's 16-lane row) * b for k < N
template <int N>
DEV void dpp_axpy(float* A, float c, float b) {
  static_assert(N == 4 || N == 8 || N == 12 || N == 16, "blocks of four");
  if constexpr (N == 4) asm("s_nop 1\n" MJH_AX4 : MJH_O4 : [c] "v"(c), [b] "v"(b));
  if constexpr (N == 8) asm("s_nop 1\n" MJH_AX8 : MJH_O8 : [c] "v"(c), [b] "v"(b));
  if constexpr (N == 12) asm("s_nop 1\n" MJH_AX12 : MJH_O12 : [c] "v"(c), [b] "v"(b));
  if constexpr (N == 16) asm("s_nop 1\n" MJH_AX16 : MJH_O16 : [c] "v"(c), [b] "v"(b));
}
#define MJH_DT(d, k) "v_fmac_f32_dpp %0, %[c], %" #d " row_newbcast:" #k " row_mask:0xf bank_mask:0xf\n"
#define MJH_DT4 MJH_DT(1, 0) MJH_DT(2, 1) MJH_DT(3, 2) MJH_DT(4, 3)
#define MJH_DT12 MJH_DT4 MJH_DT(5, 4) MJH_DT(6, 5) MJH_DT(7, 6) MJH_DT(8, 7) MJH_DT(9, 8) \
    MJH_DT(10, 9) MJH_DT(11, 10) MJH_DT(12, 11)
#define MJH_DT16 MJH_DT12 MJH_DT(13, 12) MJH_DT(14, 13) MJH_DT(15, 14) MJH_DT(16, 15)
#define MJH_I4 "v"(A[0]), "v"(A[1]), "v"(A[2]), "v"(A[3])
#define MJH_I12 MJH_I4, "v"(A[4]), "v"(A[5]), "v"(A[6]), "v"(A[7]), "v"(A[8]), "v"(A[9]), \
    "v"(A[10]), "v"(A[11])
#define MJH_I16 MJH_I12, "v"(A[12]), "v"(A[13]), "v"(A[14]), "v"(A[15])
// v + sum over k < N of (lane k of c's 16-lane row) * A[k], in k order
template <int N>
DEV float dpp_dot(float v, float c, const float* A) {
  static_assert(N == 4 || N == 12 || N == 16, "the blocks of 20, 28 and 16 or 32 entries");
  if constexpr (N == 4) asm("s_nop 1\n" MJH_DT4 "s_nop 1" : "+v"(v) : MJH_I4, [c] "v"(c));
  if constexpr (N == 12) asm("s_nop 1\n" MJH_DT12 "s_nop 1" : "+v"(v) : MJH_I12, [c] "v"(c));
  if constexpr (N == 16) asm("s_nop 1\n" MJH_DT16 "s_nop 1" : "+v"(v) : MJH_I16, [c] "v"(c));
  return v;
}
#undef MJH_AX
#undef MJH_AX4
#undef MJH_AX8
#undef MJH_AX12
#undef MJH_AX16
#undef MJH_O4
#undef MJH_O8
#undef MJH_O12
#undef MJH_O16
#undef MJH_DT
#undef MJH_DT4
#undef MJH_DT12
#undef MJH_DT16
#undef MJH_I4
#undef MJH_I12
#undef MJH_I16

// dp += sum over the four rows k = B .. B + 3 of (lane k of ds) * min(0, (lane k of e) +
// br (lane k of s)): the contribution of four one-sided constraint rows to the line
// search's slope at br
#define MJH_SL(n, k)                                                                   \
  "v_mov_b32_dpp %[t" #n "], %[e] row_newbcast:" k " row_mask:0xf bank_mask:0xf\n"
#define MJH_SM(n, k)                                                                   \
  "v_fmac_f32_dpp %[t" #n "], %[s], %[br] row_newbcast:" k " row_mask:0xf bank_mask:0xf\n"
#define MJH_SN(n) "v_min_f32 %[t" #n "], 0, %[t" #n "]\n"
#define MJH_SO(n, k)                                                                   \
  "v_fmac_f32_dpp %[dp], %[ds], %[t" #n "] row_newbcast:" k " row_mask:0xf bank_mask:0xf\n"
#define MJH_SLOPE4(a, b, c, d)                                                          \
  asm("s_nop 1\n" MJH_SL(0, a) MJH_SL(1, b) MJH_SL(2, c) MJH_SL(3, d) MJH_SM(0, a)       \
      MJH_SM(1, b) MJH_SM(2, c) MJH_SM(3, d) MJH_SN(0) MJH_SN(1) MJH_SN(2) MJH_SN(3)     \
      MJH_SO(0, a) MJH_SO(1, b) MJH_SO(2, c) MJH_SO(3, d)                                \
      : [dp] "+v"(dp), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)    \
      : [e] "v"(e), [s] "v"(s), [ds] "v"(ds), [br] "v"(br))
template <int B>
DEV float dpp_slope4(float dp, float e, float s, float ds, float br) {
  static_assert(B == 0 || B == 4 || B == 8 || B == 12, "four rows of a 16-lane row");
  float t0, t1, t2, t3;
  if constexpr (B == 0) MJH_SLOPE4("0", "1", "2", "3");
  if constexpr (B == 4) MJH_SLOPE4("4", "5", "6", "7");
  if constexpr (B == 8) MJH_SLOPE4("8", "9", "10", "11");
  if constexpr (B == 12) MJH_SLOPE4("12", "13", "14", "15");
  return dp;
}
#undef MJH_SN
#undef MJH_SLOPE4

// The same for rows with bounds of their own: dp += sum of (lane k of s) * clamp((lane k of D) *
// ((lane k of e) + br (lane k of s)), lane k of lo, lane k of hi), the upper bound first, so that
// a one-sided row (lo = -inf, hi = 0) whose breakpoint's product is no number adds nothing
#define MJH_SP(n, k)                                                                   \
  "v_mul_f32_dpp %[t" #n "], %[D], %[t" #n "] row_newbcast:" k " row_mask:0xf bank_mask:0xf\n"
#define MJH_SQ(n, k)                                                                   \
  "v_min_f32_dpp %[t" #n "], %[hi], %[t" #n "] row_newbcast:" k " row_mask:0xf bank_mask:0xf\n"
#define MJH_SR(n, k)                                                                   \
  "v_max_f32_dpp %[t" #n "], %[lo], %[t" #n "] row_newbcast:" k " row_mask:0xf bank_mask:0xf\n"
#define MJH_CLAMP4(a, b, c, d)                                                          \
  asm("s_nop 1\n" MJH_SL(0, a) MJH_SL(1, b) MJH_SL(2, c) MJH_SL(3, d) MJH_SM(0, a)       \
      MJH_SM(1, b) MJH_SM(2, c) MJH_SM(3, d) MJH_SP(0, a) MJH_SP(1, b) MJH_SP(2, c)       \
      MJH_SP(3, d) MJH_SQ(0, a) MJH_SQ(1, b) MJH_SQ(2, c) MJH_SQ(3, d) MJH_SR(0, a)       \
      MJH_SR(1, b) MJH_SR(2, c) MJH_SR(3, d) MJH_SO(0, a) MJH_SO(1, b) MJH_SO(2, c)       \
      MJH_SO(3, d)                                                                      \
      : [dp] "+v"(dp), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3)    \
      : [e] "v"(e), [s] "v"(s), [ds] "v"(s), [D] "v"(D), [lo] "v"(lo), [hi] "v"(hi),     \
        [br] "v"(br))
template <int B>
DEV float dpp_clamp4(float dp, float e, float s, float D, float lo, float hi, float br) {
  static_assert(B == 0 || B == 4 || B == 8 || B == 12, "four rows of a 16-lane row");
  float t0, t1, t2, t3;
  if constexpr (B == 0) MJH_CLAMP4("0", "1", "2", "3");
  if constexpr (B == 4) MJH_CLAMP4("4", "5", "6", "7");
  if constexpr (B == 8) MJH_CLAMP4("8", "9", "10", "11");
  if constexpr (B == 12) MJH_CLAMP4("12", "13", "14", "15");
  return dp;
}
#undef MJH_SL
#undef MJH_SM
#undef MJH_SO
#undef MJH_SP
#undef MJH_SQ
#undef MJH_SR
#undef MJH_CLAMP4

// v + (lane B of z) n + (lane B + 1 of z) a + (lane B + 2 of z) b: a contact's frame weights,
// on its quad's lanes, times its frame rows' entries
#define MJH_QUAD3(b0, b1, b2)                                                               \
  asm("s_nop 1\n"                                                                           \
      "v_fmac_f32_dpp %[v], %[z], %[n] row_newbcast:" b0 " row_mask:0xf bank_mask:0xf\n"    \
      "v_fmac_f32_dpp %[v], %[z], %[a] row_newbcast:" b1 " row_mask:0xf bank_mask:0xf\n"    \
      "v_fmac_f32_dpp %[v], %[z], %[b] row_newbcast:" b2 " row_mask:0xf bank_mask:0xf\n"    \
      "s_nop 1"                                                                              \
      : [v] "+v"(v) : [z] "v"(z), [n] "v"(n), [a] "v"(a), [b] "v"(b))
template <int B>
DEV float dpp_quad3(float v, float z, float n, float a, float b) {
  static_assert(B == 0 || B == 4 || B == 8 || B == 12, "a quad of a 16-lane row");
  if constexpr (B == 0) MJH_QUAD3("0", "1", "2");
  if constexpr (B == 4) MJH_QUAD3("4", "5", "6");
  if constexpr (B == 8) MJH_QUAD3("8", "9", "10");
  if constexpr (B == 12) MJH_QUAD3("12", "13", "14");
  return v;
}
#undef MJH_QUAD3
// rows of P = J3^T C for a contact's frame rows (n, a, b): C = [[all, d0, d2], [d0, s0, 0],
// [d2, 0, s2]], its entries on lanes B (all, d0, s0) and B + 2 (d2, s2)
#define MJH_FRAME(b0, b2)                                                                     \
  asm("s_nop 1\n"                                                                             \
      "v_mul_f32_dpp %[pn], %[all], %[n] row_newbcast:" b0 " row_mask:0xf bank_mask:0xf\n"    \
      "v_mul_f32_dpp %[pa], %[d], %[n] row_newbcast:" b0 " row_mask:0xf bank_mask:0xf\n"      \
      "v_mul_f32_dpp %[pb], %[d], %[n] row_newbcast:" b2 " row_mask:0xf bank_mask:0xf\n"      \
      "v_fmac_f32_dpp %[pn], %[d], %[a] row_newbcast:" b0 " row_mask:0xf bank_mask:0xf\n"     \
      "v_fmac_f32_dpp %[pa], %[s], %[a] row_newbcast:" b0 " row_mask:0xf bank_mask:0xf\n"     \
      "v_fmac_f32_dpp %[pb], %[s], %[b] row_newbcast:" b2 " row_mask:0xf bank_mask:0xf\n"     \
      "v_fmac_f32_dpp %[pn], %[d], %[b] row_newbcast:" b2 " row_mask:0xf bank_mask:0xf\n"     \
      "s_nop 1"                                                                               \
      : [pn] "=&v"(pn), [pa] "=&v"(pa), [pb] "=&v"(pb)                                        \
      : [all] "v"(all), [d] "v"(d), [s] "v"(s), [n] "v"(n), [a] "v"(a), [b] "v"(b))
template <int B>
DEV void dpp_frame(float all, float d, float s, float n, float a, float b, float& pn, float& pa,
                   float& pb) {
  static_assert(B == 0 || B == 4 || B == 8 || B == 12, "a quad of a 16-lane row");
  if constexpr (B == 0) MJH_FRAME("0", "2");
  if constexpr (B == 4) MJH_FRAME("4", "6");
  if constexpr (B == 8) MJH_FRAME("8", "10");
  if constexpr (B == 12) MJH_FRAME("12", "14");
}
#undef MJH_FRAME

// lane k of v's 16-lane row, on every lane of that row
template <int K>
DEV float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xF, 0xF, true));
}
// quad permutation: lane l takes v of lane (l & ~3) + (CTRL >> 2 (l & 3) & 3)
template <int CTRL>
DEV float quad_perm(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;

struct Pair {
  float a, b;
};
// lower 16-lane rows of x in every row pair (a), and the upper ones (b): x's rows 0, 2
// replicated over rows (0, 1), (2, 3), and its rows 1, 3
DEV Pair swap16(float x) {
  const unsigned u = (unsigned)__float_as_int(x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return {__int_as_float((int)r[0]), __int_as_float((int)r[1])};
}
// (x's lower half, y's lower half) and (x's upper half, y's upper half)
DEV Pair swap32(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap((unsigned)__float_as_int(x),
                                                  (unsigned)__float_as_int(y), false, false);
  return {__int_as_float((int)r[0]), __int_as_float((int)r[1])};
}
// a dof vector's 16-lane rows replicated over the team: entries 0..15 in a, 16..31 in b
template <int T>
DEV Pair rep_dof(float x) {
  if constexpr (T == 16) {
    asm("s_nop 1" : "+v"(x));  // (x may come straight out of a block, into a DPP read)
    return {x, 0.f};
  } else {
    return swap16(x);
  }
}

// ------------------------------------------------- rows of a symmetric matrix, one per lane
// NB is the padded row length (16, 20 or 28: blocks of 16 and 4 or 12), nv the length in use.
// Entries past nv are zero.

// v + (row A) . x, x replicated by rep_dof
template <int NB>
DEV float row_dot(const float* A, const Pair& x, float v = 0.f) {
  v = dpp_dot<16>(v, x.a, A);
  if constexpr (NB > 16) v = dpp_dot<NB - 16>(v, x.b, A + 16);
  return v;
}
// the row's entries below K, in blocks of four: A[j] += x_j b
template <int NB, int K>
DEV void row_axpy(float* A, const Pair& x, float b) {
  constexpr int lo = K >= 16 ? 16 : (K + 3) / 4 * 4;
  if constexpr (lo > 0) dpp_axpy<lo>(A, x.a, b);
  if constexpr (K > 16) dpp_axpy<(K - 16 + 3) / 4 * 4>(A + 16, x.b, b);
}

// shortest row that a padded length serves (the host picks the smallest that fits)
template <int NB>
constexpr int min_nv() {
  return NB == 28 ? 21 : NB == 20 ? 17 : 1;
}

// Gauss-Jordan elimination, last dof first (a tree's leaves: the light links are eliminated
// from the heavy root's rows, not the other way round, which keeps FP32 digits).  While a
// dof is not yet eliminated the remaining matrix is symmetric, so pivot row k's entry j is
// also entry (j, k), on lane j in register A[k]: one register replicated over the team
// carries the whole pivot row, and each entry's update is one broadcast multiply-add.
// Eliminating the rows above the pivot as well costs nothing (their lanes would idle) and
// leaves the solution without a back substitution.
// Returns this lane's entry of A^-1 b; A is destroyed.  ok: every pivot was positive.
template <int T, int NB, int K>
DEV void gj_solve_pivot(float* A, int nv, int i, float& b, float& rd, bool& ok) {
  if (K < min_nv<NB>() || K < nv) {  // (nv is uniform)
    const Pair c = rep_dof<T>(A[K]);
    const float p = row_bcast<(K & 15)>(K < 16 ? c.a : c.b);
    ok = ok && p > 0.f;
    const float r = __builtin_amdgcn_rcpf(p);
    const float nl = i == K ? 0.f : -(A[K] * r);
    const Pair bb = rep_dof<T>(b);
    b += row_bcast<(K & 15)>(K < 16 ? bb.a : bb.b) * nl;
    row_axpy<NB, K>(A, c, nl);
    rd = i == K ? r : rd;
  }
  if constexpr (K > 0) gj_solve_pivot<T, NB, K - 1>(A, nv, i, b, rd, ok);
}
template <int T, int NB>
DEV float gj_solve(float* A, int nv, int i, float b, bool& ok) {
  float rd = 0.f;
  gj_solve_pivot<T, NB, NB - 1>(A, nv, i, b, rd, ok);
  return b * rd;
}

// The same elimination carried to the inverse (the symmetric sweep operator), for 16-lane teams
// (wider ones sweep on the matrix cores, mjh_newton_reg.h): after every
// dof is swept, row i of A^-1 is -s A[.], s this lane's reciprocal pivot.  A swept row is
// kept without its factor s, so that no lane's row needs rescaling; the broadcast column
// takes it.  The right-hand side b rides along and comes out as A^-1 b with the accuracy of
// the elimination, which a product with the inverse does not reach; the inverse then serves
// further right-hand sides (refinement corrections) at one dot product each.
template <int T, int NB, int K>
DEV void sweep_pivot(float* A, float& s, int nv, int i, float& b, bool& ok) {
  if (K < min_nv<NB>() || K < nv) {
    const Pair c = rep_dof<T>(A[K] * s);
    const float p = row_bcast<(K & 15)>(K < 16 ? c.a : c.b);
    ok = ok && p > 0.f;
    const float r = __builtin_amdgcn_rcpf(p);
    const float al = A[K] * r;
    const float nl = i == K ? 0.f : -al;
    const Pair bb = rep_dof<T>(b * s);
    b += row_bcast<(K & 15)>(K < 16 ? bb.a : bb.b) * nl;
    row_axpy<NB, NB>(A, c, nl);
    A[K] = i == K ? -1.f : al;
    s = i == K ? r : s;
  }
  if constexpr (K > 0) sweep_pivot<T, NB, K - 1>(A, s, nv, i, b, ok);
}
template <int T, int NB>
DEV float sweep_inverse(float* A, float& s, int nv, int i, float b, bool& ok) {
  s = 1.f;
  sweep_pivot<T, NB, NB - 1>(A, s, nv, i, b, ok);
  return b * s;
}

}  // namespace mjh
