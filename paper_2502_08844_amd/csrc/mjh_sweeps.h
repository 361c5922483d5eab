// The tree sweeps with one body per lane (and one dof, one joint per lane where those are the
// parallel axis): actuation, forward_sweep and backward_and_mass, phase by phase the same
// arithmetic, for worlds of at most T bodies besides the world's.
//
// The level-parallel loops are serial chains: per level they loaded a body's number, then its
// parent's and joints' numbers, then their constants (an L1 hit each, some 500 cycles with one
// wavefront on a SIMD), and evaluated sines.  Here a lane keeps one body for the whole sweep, so
// its constants arrive in one batch as a packed record (kBodyRec), every joint's rotation is
// formed before the first level, and a level only composes rotations and adds velocities.  The
// controls, which come from HBM, are loaded before the levels and used after them.  64 quadrupeds:
// 28 thousand clocks of a step's 96 in these phases before, 19 of 87 now.
#pragma once

namespace mjh {

DEV void sweeps_lanes(const DevModel& m, float* W, const Team& t, const float* ctrl,
                      const float* dr) {
  const int lane = t.lane, nb = m.nbody, nv = m.nv;
  const float* qpos = W + m.o_qpos;
  const float* qvel = W + m.o_qvel;
  float* xpos = W + m.o_xpos;
  float* xmat = W + m.o_xmat;
  float* cvel = W + m.o_cvel;
  float* cacc = W + m.o_cacc;
  float* cdof = W + m.o_cdof;
  // ---- constants of this lane's body and dof
  const bool body = 1 + lane < nb;
  const int4* br = (const int4*)(m.body_rec + kBodyRec * min(lane, nb - 2));
  const int4 b0 = br[0], b1 = br[1], b2 = br[2];
  const float4* bf = (const float4*)(br + 3);
  const float4 f0 = bf[0], f1 = bf[1], f2 = bf[2], f3 = bf[3], f4 = bf[4], f5 = bf[5];
  const int b = b0.x, p = b0.y, level = b0.z, nj = b0.w;
  const int qa0 = b1.x, da0 = b1.y, types = b1.z, j0 = b1.w;
  const bool dof = lane < nv;
  const float4* df = (const float4*)(m.dof_rec + kDofRec * min(lane, nv - 1));
  const float4 d0 = df[0], d1 = df[1], d2 = df[2];
  const int act = __float_as_int(d0.y);
  // ---- every joint's rotation (a free joint's: the body's) and axis, in the words of the
  // sweeps' later scratch (forces, inertias)
  float* jl = W + m.o_cfrc;
  for (int j = lane; j < m.njnt; j += t.T) {
    const int4 ji = *(const int4*)(m.jnt_rec + kJntRec * j);
    const float4 ja = *(const float4*)(m.jnt_rec + kJntRec * j + 4);
    const float ax[3] = {ja.x, ja.y, ja.z};
    float Rj[9];
    if (ji.x == JNT_FREE) {
      const float* qq = qpos + ji.y + 3;
      float q[4] = {qq[0], qq[1], qq[2], qq[3]};
      const float inv = 1.f / sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
      for (int k = 0; k < 4; k++) q[k] *= inv;
      quat_to_mat(q, Rj);
    } else if (ji.x == JNT_HINGE) {
      axis_rot(ax, qpos[ji.y], Rj);
    } else {
      for (int k = 0; k < 9; k++) Rj[k] = 0.f;
      Rj[0] = qpos[ji.y];
    }
    for (int k = 0; k < 9; k++) jl[12 * j + k] = Rj[k];
    for (int k = 0; k < 3; k++) jl[12 * j + 9 + k] = ax[k];
  }
  // the world body and the origin p0 (see forward_sweep)
  if (lane < 6) {
    cvel[lane] = 0.f;
    cacc[lane] = lane < 3 ? 0.f : -m.grav[lane - 3];
  }
  if (lane < 3)
    xpos[lane] = (m.njnt > 0 && m.jnt_type[0] == JNT_FREE) ? -qpos[m.jnt_qposadr[0] + lane] : 0.f;
  const float u0 = dof && act >= 0 && ctrl ? ctrl[act] : 0.f;
  t.sync();
  // ---- forward, level by level
  float pos[3] = {f0.x, f0.y, f0.z}, R[9], V[6], A[6];
#pragma unroll
  for (int k = 0; k < 9; k++) R[k] = 0.f;
#pragma unroll
  for (int k = 0; k < 6; k++) V[k] = A[k] = 0.f;
  for (int lv = 1; lv < m.nlevel; lv++) {
    if (body && level == lv) {
      float Rp[9];
      for (int k = 0; k < 9; k++) Rp[k] = xmat[9 * p + k];
      mv3(Rp, pos, pos);
      for (int k = 0; k < 3; k++) pos[k] += xpos[3 * p + k];
      if (m.rot_id) {
        for (int k = 0; k < 9; k++) R[k] = Rp[k];
      } else {
        const float br9[9] = {f0.w, f1.x, f1.y, f1.z, f1.w, f2.x, f2.y, f2.z, f2.w};
        mm3(Rp, br9, R);
      }
      for (int k = 0; k < 6; k++) { V[k] = cvel[6 * p + k]; A[k] = cacc[6 * p + k]; }
      int da = da0;
      for (int j = 0; j < nj; j++) {
        const float* jr = jl + 12 * (j0 + j);
        const int type = types >> (2 * j) & 3;
        float* S = cdof + 6 * da;
        float Sd[6];
        if (type == JNT_FREE) {
          for (int k = 0; k < 9; k++) R[k] = jr[k];
          for (int k = 0; k < 3; k++) pos[k] = qpos[qa0 + k] + xpos[k];  // relative to p0
          for (int i = 0; i < 3; i++) {
            float* s = S + 6 * i;
            s[0] = s[1] = s[2] = 0.f;
            s[3] = (i == 0) ? 1.f : 0.f; s[4] = (i == 1) ? 1.f : 0.f; s[5] = (i == 2) ? 1.f : 0.f;
            V[3 + i] += qvel[da + i];
          }
          float r[3][6];
          for (int i = 0; i < 3; i++) {
            const float col[3] = {R[i], R[3 + i], R[6 + i]};
            for (int k = 0; k < 3; k++) r[i][k] = col[k];
            cross3(pos, col, r[i] + 3);
            for (int k = 0; k < 6; k++) S[6 * (3 + i) + k] = r[i][k];
            for (int k = 0; k < 6; k++) V[k] += r[i][k] * qvel[da + 3 + i];
          }
          for (int i = 0; i < 3; i++) {
            crossm(V, r[i], Sd);
            for (int k = 0; k < 6; k++) A[k] += Sd[k] * qvel[da + 3 + i];
          }
          da += 6;
          continue;
        }
        float ax[3] = {jr[9], jr[10], jr[11]}, s[6];
        if (type == JNT_SLIDE) {
          mv3(R, ax, ax);
          for (int k = 0; k < 3; k++) pos[k] += ax[k] * jr[0];
          s[0] = s[1] = s[2] = 0.f;
          s[3] = ax[0]; s[4] = ax[1]; s[5] = ax[2];
        } else {  // hinge: R Rot(a, q) (see forward_sweep)
          float anc[3] = {pos[0], pos[1], pos[2]}, off[3], Rj[9];
          float jp[3] = {0.f, 0.f, 0.f};
          if (!m.jpos0) {
            const float* q = m.jnt_pos + 3 * (j0 + j);
            for (int k = 0; k < 3; k++) jp[k] = q[k];
            mv3(R, jp, off);
            for (int k = 0; k < 3; k++) anc[k] = pos[k] + off[k];
          }
          for (int k = 0; k < 9; k++) Rj[k] = jr[k];
          mm3(R, Rj, R);
          mv3(R, ax, ax);
          if (!m.jpos0) {
            mv3(R, jp, off);
            for (int k = 0; k < 3; k++) pos[k] = anc[k] - off[k];
          }
          s[0] = ax[0]; s[1] = ax[1]; s[2] = ax[2];
          cross3(anc, ax, s + 3);
        }
        const float qd = qvel[da];
        for (int k = 0; k < 6; k++) {
          S[k] = s[k];
          V[k] += s[k] * qd;
        }
        crossm(V, s, Sd);
        for (int k = 0; k < 6; k++) A[k] += Sd[k] * qd;
        da++;
      }
      for (int k = 0; k < 3; k++) xpos[3 * b + k] = pos[k];
      for (int k = 0; k < 9; k++) xmat[9 * b + k] = R[k];
      for (int k = 0; k < 6; k++) { cvel[6 * b + k] = V[k]; cacc[6 * b + k] = A[k]; }
    }
    t.sync();
  }
  // ---- actuation (actuation())
  float frc = 0.f;
  if (dof) {
    frc = -d0.x * qvel[lane];
    if (act >= 0) {
      const float u = fminf(fmaxf(u0, d1.z), d1.w);
      if (__float_as_int(d0.z) == ACT_MOTOR) {
        frc += d0.w * u;
      } else {
        float kp = d1.x, kd = d1.y, q0 = d2.x;
        if (dr) {
          kp *= dr[kDrKp];
          kd *= dr[kDrKd];
          q0 -= dr[kDrHead + act];
        }
        frc += kp * (q0 + d0.w * u - qpos[__float_as_int(d2.y)]) - kd * qvel[lane];
      }
    }
  }
  // ---- spatial inertia and bias force of this lane's body (see forward_sweep)
  float* cfrc = W + m.o_cfrc;
  float* Ic = W + m.o_cinert;
  float ic[kCinert], fb[6];
#pragma unroll
  for (int k = 0; k < kCinert; k++) ic[k] = 0.f;
#pragma unroll
  for (int k = 0; k < 6; k++) fb[k] = 0.f;
  if (body) {
    float c[3], RI[9], ip[3] = {f3.y, f3.z, f3.w};
    float mass = f3.x;
    if (dr && b == 1) {
      for (int k = 0; k < 3; k++) ip[k] += dr[kDrCom + k];
      mass += dr[kDrPayload];
    }
    mv3(R, ip, c);
    for (int k = 0; k < 3; k++) c[k] += pos[k];
    const float Il[9] = {f4.x, f4.w, f5.x, f4.w, f4.y, f5.y, f5.x, f5.y, f4.z};
    mm3(R, Il, RI);
    auto iw = [&](int i, int j) {
      return RI[3 * i] * R[3 * j] + RI[3 * i + 1] * R[3 * j + 1] + RI[3 * i + 2] * R[3 * j + 2];
    };
    const float cc = dot3(c, c);
    ic[0] = mass;
    ic[1] = mass * c[0]; ic[2] = mass * c[1]; ic[3] = mass * c[2];
    ic[4] = iw(0, 0) + mass * (cc - c[0] * c[0]);
    ic[5] = iw(1, 1) + mass * (cc - c[1] * c[1]);
    ic[6] = iw(2, 2) + mass * (cc - c[2] * c[2]);
    ic[7] = iw(0, 1) - mass * c[0] * c[1];
    ic[8] = iw(0, 2) - mass * c[0] * c[2];
    ic[9] = iw(1, 2) - mass * c[1] * c[2];
    float IA[6], IV[6], VIV[6];
    inertia_mul(ic, A, IA);
    inertia_mul(ic, V, IV);
    crossf(V, IV, VIV);
    for (int k = 0; k < 6; k++) fb[k] = IA[k] + VIV[k];
    for (int k = 0; k < kCinert; k++) Ic[kCinert * b + k] = ic[k];
    for (int k = 0; k < 6; k++) cfrc[6 * b + k] = fb[k];
  }
  // the mass matrix's entries of this lane (the first kPairs), loaded ahead of the levels
  constexpr int kPairs = 4;
  int pr[kPairs];
#pragma unroll
  for (int q = 0; q < kPairs; q++) {
    const int k = lane + q * t.T;
    pr[q] = k < m.nmpair ? m.mpair[k] : -1;
  }
  t.sync();
  // ---- backward, level by level: subtree inertias and forces
  const int nch = b2.x;
  for (int lv = m.nlevel - 2; lv >= 1; lv--) {
    if (body && level == lv && nch > 0) {
      for (int c = 0; c < nch; c++) {
        const int ch = c < 4 ? (b2.y >> (8 * c) & 255) : m.child_list[b2.z + c];
        for (int k = 0; k < kCinert; k++) ic[k] += Ic[kCinert * ch + k];
        for (int k = 0; k < 6; k++) fb[k] += cfrc[6 * ch + k];
      }
      for (int k = 0; k < kCinert; k++) Ic[kCinert * b + k] = ic[k];
      for (int k = 0; k < 6; k++) cfrc[6 * b + k] = fb[k];
    }
    t.sync();
  }
  // ---- bias force c_i = S_i . f_subtree; F_i = Ic S_i; the armatures in a0's words, still free
  float* F = W + m.o_F;
  if (dof) {
    const int db = __float_as_int(d2.w);
    W[m.o_frc + lane] = frc - dot6(cdof + 6 * lane, cfrc + 6 * db);
    inertia_mul(Ic + kCinert * db, cdof + 6 * lane, F + 6 * lane);
    W[m.o_a0 + lane] = (dr && lane >= 6) ? dr[kDrHead + m.nu + lane - 6] : d2.z;
  }
  t.sync();
  // ---- M_ij = S_j . F_i for j ancestor-or-self of i
  float* M = W + m.o_M;
  auto entry = [&](int pk) {
    const int i = pk >> 16, j = pk & 0xffff;
    float v = dot6(cdof + 6 * j, F + 6 * i);
    if (i == j) v += W[m.o_a0 + i];
    M[tri(i, j)] = v;
  };
#pragma unroll
  for (int q = 0; q < kPairs; q++)
    if (pr[q] >= 0) entry(pr[q]);
  for (int k = lane + kPairs * t.T; k < m.nmpair; k += t.T) entry(m.mpair[k]);
  t.sync();
}

}  // namespace mjh
