// Per-tile evaluation of the 3D particle response (Eq. 11) shared by the
// forward and backward compositing kernels.
//
// Conditioning.  A particle's response along a pixel ray depends on
// omega^2 = |o_g x d_g|^2 / |d_g|^2 with o_g = S^-1 R^T (o - mu) and
// d_g = S^-1 R^T d.  For a small particle far from the camera, o_g is long
// (distance / scale, up to ~1e4) and nearly parallel to d_g, so forming the
// cross product from FP32 rays loses most of its bits.  Instead each tile gets
// an FP64 frame (origin o_T, unit anchor direction n, tangent basis e1, e2)
// and every pixel ray is written EXACTLY as a direction proportional to
// n + u e1 + v e2 (u, v small, so FP32 holds them to ~1e-10), plus, under a
// rolling shutter, an origin o_T + dt (c1 - c0).  Per (tile, particle) pair
// the kernel forms in FP64, once,
//   d_g(n), d_g(e1), d_g(e2), w = o_g x d_g(n), A = o_g x d_g(e1),
//   B = o_g x d_g(e2)   (and the dt terms m x ...,  m = S^-1 R^T (c1 - c0))
// and stores them as FP32; per pixel the cross product is the short sum
// w + u A + v B whose terms are of the size of the result, so FP32 keeps
// ~1e-6 relative accuracy for every particle.  This costs fewer FP32 ops per
// evaluation than transforming each ray into the particle frame.
//
// The same inline functions, with explicit fmaf and contraction disabled at
// compile time, are used by forward and backward so that every discrete
// decision (tau_max > 0, alpha >= alpha_min, clamping) is identical in both.
#pragma once
#include "common.h"

namespace gut {

// FP64 tile frame kept in LDS: origin, anchor direction, tangent basis, time.
struct TileFrameD {
  double o[3], n[3], e1[3], e2[3], tT;
  float umax, vmax, dtmax, l2amin;  // compositing: the tile's |u|, |v|, |dt| bounds and log2(alpha_min)
};

__device__ inline void tile_frame(const DevCam& cam, int tx, int ty, TileFrameD* F) {
  double ua = fmin(tx * (double)kTile + 0.5 * kTile, (double)cam.W);
  double va = fmin(ty * (double)kTile + 0.5 * kTile, (double)cam.H);
  int ra = min(ty * kTile + kTile / 2, cam.H - 1);
  double tT = row_time(cam, ra);
  bool ok;
  d3 dca = unproject_dir(cam, ua, va, &ok);
  d3 o, d;
  ray_at(cam, tT, dca, &o, &d);
  d = scl(d, 1.0 / sqrt(dot(d, d)));
  d3 ref = fabs(d.x) <= fabs(d.y) && fabs(d.x) <= fabs(d.z) ? mk3(1, 0, 0)
           : (fabs(d.y) <= fabs(d.z) ? mk3(0, 1, 0) : mk3(0, 0, 1));
  d3 e1 = cross(d, ref);
  e1 = scl(e1, 1.0 / sqrt(dot(e1, e1)));
  d3 e2 = cross(d, e1);
  F->o[0] = o.x; F->o[1] = o.y; F->o[2] = o.z;
  F->n[0] = d.x; F->n[1] = d.y; F->n[2] = d.z;
  F->e1[0] = e1.x; F->e1[1] = e1.y; F->e1[2] = e1.z;
  F->e2[0] = e2.x; F->e2[1] = e2.y; F->e2[2] = e2.z;
  F->tT = tT;
}

// Pixel ray in tile coordinates: direction ~ n + u e1 + v e2, origin o_T + dt (c1 - c0).
__device__ inline bool pixel_ray(const DevCam& cam, const TileFrameD& F, int px, int py, float* u,
                                 float* v, float* dt) {
  double tr = row_time(cam, py);
  bool valid;
  d3 dc = unproject_dir(cam, px + 0.5, py + 0.5, &valid);
  d3 o, d;
  ray_at(cam, tr, dc, &o, &d);
  double dn = dot(d, mk3(F.n[0], F.n[1], F.n[2]));
  if (!(dn > 0.0)) return false;
  double idn = 1.0 / dn;
  *u = (float)(dot(d, mk3(F.e1[0], F.e1[1], F.e1[2])) * idn);
  *v = (float)(dot(d, mk3(F.e2[0], F.e2[1], F.e2[2])) * idn);
  *dt = (float)(tr - F.tT);
  return valid;
}

// log2(e) / 2: omega^2 / 2 in natural units is omega^2 * kHalfLog2e in log2 units.
constexpr double kHalfLog2e = 0.72134752044448170368;

// Pair slots (float4 each) kept in LDS for one (tile, particle) pair.
//
// Global shutter.  The two quadratic forms of a pixel's (u, v) that decide
// the response are factored in FP64 (QR of the affine maps (u, v) -> vector)
// into sums of squares,
//   |o_g x d_g|^2 log2(e)/2 = (f1 + r11 u + r12 v)^2 + (f2 + r22 v)^2 + f3
//   |d_g|^2                 = (g1 + h11 u + h12 v)^2 + (g2 + h22 v)^2 + g3
// so a pixel needs 10 FMAs for both and no term cancels beyond what the
// affine maps themselves carry.
//   0: f1 r11 r12 Kp    1: f2 r22 f3 lsig    2: g1 h11 h12 E11
//   3: g2 h22 g3 E12    4: colour r g (FP64)  5: s ta tb E22
//   6: colour b (FP64), uc vc
// and, for the backward only, the vectors for the closest point p:
//   7: d_g(n).xyz w.x   8: d_g(e1).xyz w.y   9: d_g(e2).xyz w.z
//  10: A.xyz B.x       11: B.y B.z - -
// Rolling shutter.  The origin moves with the row, so the cross product is
// bilinear in (u, v) and dt and is formed from its vectors per pixel:
//   0: d_g(n).xyz E11    1: d_g(e1).xyz lsig  2: d_g(e2).xyz Kp
//   3: w.xyz ta          4: A.xyz tb          5: B.xyz s
//   6: colour r g (FP64) 7: (m x d_g(n)).xyz m.d_g(n)
//   8: (m x d_g(e1)).xyz m.d_g(e1)               9: (m x d_g(e2)).xyz m.d_g(e2)
//  10: colour b (FP64), uc vc  11: E12 E22 - -
// (colours are kept in FP64 because the compositing accumulates in FP64)
// Here w = o_g x d_g(n), A = o_g x d_g(e1), B = o_g x d_g(e2),
// s, ta, tb = o_g . d_g(.) (the tau_max > 0 test, needed per pixel only when
// its sign varies over the tile: then E11 carries a minus sign), lsig = log2(sigma) and
// Kp = log2(sigma / alpha_min) (-1: never contributes), so that
//   alpha = min(2^(lsig - omega'^2), alpha_max),  alpha >= alpha_min <=> omega'^2 <= Kp
// with omega'^2 = omega^2 log2(e) / 2.  E11, E12, E22 and (uc, vc) are the
// culling ellipse's matrix, scaled so that it reads E11 x^2 + 2 E12 xy + E22
// y^2 <= 1, and its centre, for build_lists (E = 0: no culling).
// Bit of pair_setup's result set when the sign of o_g . d_g varies over the
// tile (the per-pixel tau_max > 0 test is needed); the low bits are per quadrant.
constexpr unsigned kMixedBit = 1u << 8;

template <bool RS, bool BWD>
struct Slots {
  static constexpr int N = RS ? 12 : (BWD ? 12 : 7);
};

// 1 / sqrt(x) for a normal x > 0: the hardware estimate (relative error
// below 2^-22) and one Newton step, ~1e-13 relative: the factorisation below
// needs ~1e-7.
__device__ __forceinline__ double rsq64(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// QR of the affine map (u, v) -> c0 + u c1 + v c2 (FP64 Gram-Schmidt; one
// pass keeps the form to ~1e-7 of the alpha_min decision scale, below the
// FP32 rounding the coefficients then take): |c0 + u c1 + v c2|^2 =
// (q[0] + q[1] u + q[2] v)^2 + (q[3] + q[4] v)^2 + q[5].
__device__ inline void affine_qr(d3 c0, d3 c1, d3 c2, double q[6]) {
  // (a norm below 1e-300 counts as zero: the estimate is not made for denormals)
  const double n11 = dot(c1, c1), i11 = n11 > 1e-300 ? rsq64(n11) : 0.0;
  const double r11 = n11 * i11;
  const d3 a1 = scl(c1, i11);
  const double r12 = dot(c2, a1);
  const d3 b = axpy(-r12, a1, c2);
  const double n22 = dot(b, b), i22 = n22 > 1e-300 ? rsq64(n22) : 0.0;
  const double r22 = n22 * i22;
  const d3 a2 = scl(b, i22);
  const double f1 = dot(c0, a1), f2 = dot(c0, a2);
  const d3 rem = axpy(-f2, a2, axpy(-f1, a1, c0));
  q[0] = f1; q[1] = r11; q[2] = r12; q[3] = f2; q[4] = r22; q[5] = dot(rem, rem);
}

// Per-wave culling.  With d_g = D x, D = [d_g(n) d_g(e1) d_g(e2)],
// x = (1, u, v), the pixels where omega^2 <= K' form {x : x^T N x <= 0} with
// N_ij = (o_g x D_i).(o_g x D_j) - K' D_i.D_j  (Lagrange's identity on
// |o_g|^2 |d_g|^2 - (o_g.d_g)^2 - K' |d_g|^2), i.e. an ellipse in (u, v)
// that is tested exactly against the pixel box of each quadrant of the tile
// (8 x 8 pixels; quadrant k = column + 2 row).  K' carries a 1e-3
// relative margin (and, under a rolling shutter, the distance the ray origin
// moves within the tile, which bounds how far the line moves), so a culled
// pair fails the per-pixel FP32 test for every pixel of the quadrant (that
// test's own rounding is ~1e-6 relative) and culling changes no result.
// Forward and backward cull identically.
struct QuadBoxes {
  float u0[4], u1[4], v0[4], v1[4];
  float cmax[4];  // largest clip distance of the quadrant's pixels (hybrid rendering)
};

// Does the ellipse qmin + [du dv] [[N11 N12] [N12 N22]] [du dv]^T <= 0
// (qmin < 0, matrix positive definite; coordinates relative to its centre)
// meet the box [a0, a1] x [b0, b1]?  The quadratic is convex, so its minimum
// over the box is at the centre if the centre is inside, else on an edge that
// faces the centre, where it is a 1D quadratic minimised in closed form and
// clamped.  (x, y) below is the box's point nearest the centre: the line at x
// is the facing vertical edge, or runs through the box's inside if there is
// none, and likewise the line at y.
__device__ inline bool ellipse_meets_box(double qmin, double N11, double N12, double N22,
                                         double iN11, double iN22, double a0, double a1,
                                         double b0, double b1) {
  const double slack = -1e-6 * qmin;
  const double x = fmin(fmax(0.0, a0), a1), y = fmin(fmax(0.0, b0), b1);
  const double ye = fmin(fmax(-N12 * x * iN22, b0), b1), xe = fmin(fmax(-N12 * y * iN11, a0), a1);
  const double qx = fma(N22 * ye, ye, fma(2.0 * N12 * x, ye, fma(N11 * x, x, qmin)));
  const double qy = fma(N11 * xe, xe, fma(2.0 * N12 * y, xe, fma(N22 * y, y, qmin)));
  return (qx <= slack) | (qy <= slack);
}

// Forms a pair's slots (FP64 -> FP32) and returns one bit per quadrant: bit k
// set when quadrant k's pixel box may see alpha >= alpha_min.  GEN:
// the response has degree th.kdeg > 2, and the threshold kept in Kp is the
// one on omega'^2 where the degree-n exponent reaches log2(sigma / alpha_min).
// CLIP (hybrid rendering): a quadrant whose largest clip distance (wb.cmax) lies
// before the particle's alpha_min ellipsoid loses its bit too -- every hit it
// could see would be clipped.
template <bool RS, bool BWD, bool GEN, bool CLIP>
__device__ inline unsigned pair_setup(const float4* __restrict__ record,
                                      const float* __restrict__ rgb, long long e, int i,
                                      const TileFrameD& F, const DevCam& cam, float umax,
                                      float vmax, float dtmax, const Thresholds& th,
                                      float log2_amin, const QuadBoxes& wb, float4* out) {
  const float amin = th.alpha_min;
  float4 r0 = record[4 * (long long)i], r1 = record[4 * (long long)i + 1];
  float4 r2 = record[4 * (long long)i + 2], r3 = record[4 * (long long)i + 3];
  const double M[9] = {r1.x, r1.y, r1.z, r2.x, r2.y, r2.z, r3.x, r3.y, r3.z};
  d3 rel = mk3(F.o[0] - (double)r0.x, F.o[1] - (double)r0.y, F.o[2] - (double)r0.z);
  d3 og = mv(M, rel);
  d3 dn = mv(M, mk3(F.n[0], F.n[1], F.n[2]));
  d3 da = mv(M, mk3(F.e1[0], F.e1[1], F.e1[2]));
  d3 db = mv(M, mk3(F.e2[0], F.e2[1], F.e2[2]));
  d3 w = cross(og, dn), A = cross(og, da), B = cross(og, db);
  double s = dot(og, dn), ta = dot(og, da), tb = dot(og, db);
  double spread = fma(umax, fabs(ta), vmax * fabs(tb));
  d3 w2 = mk3(0, 0, 0), A2 = w2, B2 = w2;
  double s2 = 0, ta2 = 0, tb2 = 0, mlen = 0;
  if (RS) {
    d3 m = mv(M, mk3(cam.dc[0], cam.dc[1], cam.dc[2]));
    w2 = cross(m, dn); A2 = cross(m, da); B2 = cross(m, db);
    s2 = dot(m, dn); ta2 = dot(m, da); tb2 = dot(m, db);
    spread = fma(dtmax, fma(umax, fabs(ta2), fma(vmax, fabs(tb2), fabs(s2))), spread);
    mlen = sqrt(dot(m, m));
  }
  const double oo = dot(og, og);
  const float sigma = r0.w;
  bool never = false, mixed = false;
  if (s + spread < 0.0) {
    // o_g . d_g < 0 (tau_max > 0) for every ray of the tile
  } else if (s - spread >= 0.0) {
    never = true;  // tau_max <= 0 for every ray
  } else {
    mixed = true;  // decide per pixel
  }
  const float lsig = log2f(sigma);
  float Kp = (!never && sigma >= amin) ? lsig - log2_amin : -1.0f;
  // degree n: 2^(k_h log2 q + k_l) <= Kp  <=>  q <= 2^((log2 Kp - k_l) / k_h)
  if (GEN && Kp > 0.0f) Kp = exp2f((log2f(Kp) - th.k_l) * th.k_inv_h);
  // the per-pixel test uses this FP32 Kp; cull with it in natural units
  double Kc = (double)Kp / kHalfLog2e * (1.0 + 1e-3) + 1e-5;
  if (RS) {
    const double r = sqrt(Kc) + dtmax * mlen * (1.0 + 1e-6);
    Kc = r * r;
  }
  // The culling ellipse's matrix N (below).  Without a rolling shutter the
  // slots' factorised forms are made first and N is read off them, so that
  // the FP64 vectors are dead before the culling: from
  // |c0 + u c1 + v c2|^2 = (q0 + q1 u + q2 v)^2 + (q3 + q4 v)^2 + q5,
  // |c0|^2 = q0^2 + q3^2 + q5, c0.c1 = q0 q1, c0.c2 = q0 q2 + q3 q4,
  // |c1|^2 = q1^2, c1.c2 = q1 q2, |c2|^2 = q2^2 + q4^2.  qc carries the
  // factor log2(e)/2, so N comes scaled by it, which leaves the ellipse.
  double N00 = 0.0, N01 = 0.0, N02 = 0.0, N11 = 0.0, N12 = 0.0, N22 = 0.0;
  if (!RS) {
    double qc[6], qd[6];
    const double sc = sqrt(kHalfLog2e);
    affine_qr(scl(w, sc), scl(A, sc), scl(B, sc), qc);
    affine_qr(dn, da, db, qd);
    out[0] = make_float4((float)qc[0], (float)qc[1], (float)qc[2], Kp);
    out[1] = make_float4((float)qc[3], (float)qc[4], (float)qc[5], lsig);
    out[2] = make_float4((float)qd[0], (float)qd[1], (float)qd[2], 0.0f);
    out[3] = make_float4((float)qd[3], (float)qd[4], (float)qd[5], 0.0f);
    out[5] = make_float4((float)s, (float)ta, (float)tb, 0.0f);
    if (BWD) {
      out[7] = make_float4((float)dn.x, (float)dn.y, (float)dn.z, (float)w.x);
      out[8] = make_float4((float)da.x, (float)da.y, (float)da.z, (float)w.y);
      out[9] = make_float4((float)db.x, (float)db.y, (float)db.z, (float)w.z);
      out[10] = make_float4((float)A.x, (float)A.y, (float)A.z, (float)B.x);
      out[11] = make_float4((float)B.y, (float)B.z, 0.0f, 0.0f);
    }
    const double K2 = Kc * kHalfLog2e;
    N00 = fma(-K2, fma(qd[0], qd[0], fma(qd[3], qd[3], qd[5])), fma(qc[0], qc[0], fma(qc[3], qc[3], qc[5])));
    N01 = fma(-K2, qd[0] * qd[1], qc[0] * qc[1]);
    N02 = fma(-K2, fma(qd[0], qd[2], qd[3] * qd[4]), fma(qc[0], qc[2], qc[3] * qc[4]));
    N11 = fma(-K2, qd[1] * qd[1], qc[1] * qc[1]);
    N12 = fma(-K2, qd[1] * qd[2], qc[1] * qc[2]);
    N22 = fma(-K2, fma(qd[2], qd[2], qd[4] * qd[4]), fma(qc[2], qc[2], qc[4] * qc[4]));
  }
  unsigned flags = 0;
  float E11 = 0.0f, E12 = 0.0f, E22 = 0.0f, ecu = 0.0f, ecv = 0.0f;
  if (Kp >= 0.0f) {
    if (oo <= Kc) {
      flags = 15u;  // the ray origin is inside the particle's alpha_min ellipsoid
    } else {
      if (RS) {
        N00 = fma(-Kc, dot(dn, dn), dot(w, w));
        N01 = fma(-Kc, dot(dn, da), dot(w, A));
        N02 = fma(-Kc, dot(dn, db), dot(w, B));
        N11 = fma(-Kc, dot(da, da), dot(A, A));
        N12 = fma(-Kc, dot(da, db), dot(A, B));
        N22 = fma(-Kc, dot(db, db), dot(B, B));
      }
      const double det = fma(N11, N22, -N12 * N12);
      if (!(N11 > 0.0) || !(N22 > 0.0) || !(det > 1e-9 * N11 * N22)) {
        flags = 15u;  // not a well-conditioned ellipse in the tile plane: no culling
      } else {
        // 1/det, 1/N11 and 1/N22 from one division
        const double p11 = N11 * N22, rq = 1.0 / (det * p11);
        const double idet = p11 * rq;
        const double uc = fma(N02, N12, -N01 * N22) * idet, vc = fma(N01, N12, -N02 * N11) * idet;
        const double qmin = fma(N02, vc, fma(N01, uc, N00));
        if (qmin < 0.0) {
          const double iN11 = det * N22 * rq, iN22 = det * N11 * rq;
          const double sc = -__builtin_amdgcn_rcp(qmin);
          E11 = (float)(N11 * sc);
          E12 = (float)(N12 * sc);
          E22 = (float)(N22 * sc);
          ecu = (float)uc;
          ecv = (float)vc;
          for (int k = 0; k < 4; k++)
            if (ellipse_meets_box(qmin, N11, N12, N22, iN11, iN22, wb.u0[k] - uc, wb.u1[k] - uc,
                                  wb.v0[k] - vc, wb.v1[k] - vc))
              flags |= 1u << k;
        }
      }
    }
  }
  if (CLIP && flags) {
    // Any accepted hit is a point of the ellipsoid |M (x - mu)|^2 <= Kc, whose
    // world radius is at most sqrt(Kc) s_max (s_k = 1 / |row k of M|), so it
    // lies at least |o - mu| - sqrt(Kc) s_max from the ray origin o, which
    // under a rolling shutter moves up to dtmax |c1 - c0| from o_T.  The
    // per-pixel test carries ~1e-6 relative error: a 1e-4 margin keeps every
    // culled pair clipped there too.
    const double Kc0 = (double)Kp / kHalfLog2e * (1.0 + 1e-3) + 1e-5;
    double rmin = 3e300;
    for (int k = 0; k < 3; k++) rmin = fmin(rmin, M[3 * k] * M[3 * k] + M[3 * k + 1] * M[3 * k + 1] +
                                                      M[3 * k + 2] * M[3 * k + 2]);
    double lb = sqrt(dot(rel, rel)) - sqrt(Kc0 / rmin);
    if (RS) lb -= (double)dtmax * sqrt(cam.dc[0] * cam.dc[0] + cam.dc[1] * cam.dc[1] + cam.dc[2] * cam.dc[2]);
    for (int k = 0; k < 4; k++)
      if (lb > (double)wb.cmax[k] * (1.0 + 1e-4)) flags &= ~(1u << k);
  }
  if (mixed && flags) {
    flags |= kMixedBit;
    E11 = -E11;  // (also -0)
  }
  const float* c = rgb + 3 * e;
  if (!RS) {
    reinterpret_cast<double2*>(out + 4)[0] = make_double2(c[0], c[1]);
    reinterpret_cast<double*>(out + 6)[0] = c[2];
    out[2].w = E11;
    out[3].w = E12;
    out[5].w = E22;
    reinterpret_cast<float2*>(out + 6)[1] = make_float2(ecu, ecv);
  } else {
    out[0] = make_float4((float)dn.x, (float)dn.y, (float)dn.z, E11);
    out[1] = make_float4((float)da.x, (float)da.y, (float)da.z, lsig);
    out[2] = make_float4((float)db.x, (float)db.y, (float)db.z, Kp);
    out[3] = make_float4((float)w.x, (float)w.y, (float)w.z, (float)ta);
    out[4] = make_float4((float)A.x, (float)A.y, (float)A.z, (float)tb);
    out[5] = make_float4((float)B.x, (float)B.y, (float)B.z, (float)s);
    reinterpret_cast<double2*>(out + 6)[0] = make_double2(c[0], c[1]);
    out[7] = make_float4((float)w2.x, (float)w2.y, (float)w2.z, (float)s2);
    out[8] = make_float4((float)A2.x, (float)A2.y, (float)A2.z, (float)ta2);
    out[9] = make_float4((float)B2.x, (float)B2.y, (float)B2.z, (float)tb2);
    reinterpret_cast<double*>(out + 10)[0] = c[2];
    reinterpret_cast<float2*>(out + 10)[1] = make_float2(ecu, ecv);
    out[11] = make_float4(E12, E22, 0.0f, 0.0f);
  }
  return flags;
}

struct Eval {
  float a;       // alpha after the alpha_max clamp
  float lq;      // degree-n responses: log2 of omega'^2
  bool clamped;  // sigma rho > alpha_max
  float cc;      // omega'^2 |d_g|^2 (omega'^2 = omega^2 log2(e) / 2); +inf: no hit (tau_max <= 0, or clipped)
  float dd;      // |d_g|^2
  float idd;     // 1 / |d_g|^2
  float araw;    // sigma rho before the alpha_max clamp
  float3 dg, cr; // rolling shutter only: d_g and o_g x d_g
};

// One pair's decision terms, loaded from LDS.
template <bool RS>
struct PairRegs {
  float4 p0, p1, p2, p3, p4, p5;
  float4 p7, p8, p9;
  float lsig, Kp, flag;  // flag: a minus sign if the sign of o_g . d_g varies over the tile
};

template <bool RS>
__device__ __forceinline__ void load_pair(const float4* P, PairRegs<RS>& r) {
  r.p0 = P[0]; r.p1 = P[1]; r.p2 = P[2]; r.p3 = P[3];
  if (RS) {
    r.p4 = P[4]; r.p5 = P[5]; r.p7 = P[7]; r.p8 = P[8]; r.p9 = P[9];
    r.lsig = r.p1.w; r.Kp = r.p2.w; r.flag = r.p0.w;
  } else {
    r.lsig = r.p1.w; r.Kp = r.p0.w; r.flag = r.p2.w;
  }
}

// Discards the hit where no is set: cc = +inf against |d_g|^2 = 1, so that
// eval_hit stays one bare compare, whatever |d_g|^2 was (a ballot of a combined
// lane flag goes through a vector register, two instructions more).
__device__ __forceinline__ void reject(bool no, Eval* o) {
  o->cc = no ? INFINITY : o->cc;
  o->dd = no ? 1.0f : o->dd;
}

// Stage 1 of the response on one pixel ray (Eq. 11): omega'^2 |d_g|^2 and
// |d_g|^2, for eval_hit's test omega'^2 <= Kp (<=> alpha >= alpha_min)
// without any transcendental (mixed: the chunk holds pairs whose tau_max sign
// varies over the tile: their hits behind the camera are discarded here).
template <bool RS>
__device__ __forceinline__ void eval_test(const PairRegs<RS>& r, const float4* P, float u, float v,
                                          float dt, bool mixed, Eval* o) {
  if (!RS) {
    const float t1 = fmaf(v, r.p0.z, fmaf(u, r.p0.y, r.p0.x));
    const float t2 = fmaf(v, r.p1.y, r.p1.x);
    o->cc = fmaf(t1, t1, fmaf(t2, t2, r.p1.z));
    const float e1 = fmaf(v, r.p2.z, fmaf(u, r.p2.y, r.p2.x));
    const float e2 = fmaf(v, r.p3.y, r.p3.x);
    o->dd = fmaf(e1, e1, fmaf(e2, e2, r.p3.z));
    if (mixed) {  // rare, and uniform across the wave
      const float4 p5 = P[5];
      const float sg = fmaf(v, p5.z, fmaf(u, p5.y, p5.x));
      reject(!(sg < 0.0f || !__builtin_signbitf(r.flag)), o);
    }
  } else {
    float3 dg = f3(fmaf(v, r.p2.x, fmaf(u, r.p1.x, r.p0.x)), fmaf(v, r.p2.y, fmaf(u, r.p1.y, r.p0.y)),
                   fmaf(v, r.p2.z, fmaf(u, r.p1.z, r.p0.z)));
    float3 cr = f3(fmaf(v, r.p5.x, fmaf(u, r.p4.x, r.p3.x)), fmaf(v, r.p5.y, fmaf(u, r.p4.y, r.p3.y)),
                   fmaf(v, r.p5.z, fmaf(u, r.p4.z, r.p3.z)));
    float3 m = f3(fmaf(v, r.p9.x, fmaf(u, r.p8.x, r.p7.x)), fmaf(v, r.p9.y, fmaf(u, r.p8.y, r.p7.y)),
                  fmaf(v, r.p9.z, fmaf(u, r.p8.z, r.p7.z)));
    cr = f3(fmaf(dt, m.x, cr.x), fmaf(dt, m.y, cr.y), fmaf(dt, m.z, cr.z));
    o->dd = fmaf(dg.z, dg.z, fmaf(dg.y, dg.y, dg.x * dg.x));
    o->cc = fmaf(cr.z, cr.z, fmaf(cr.y, cr.y, cr.x * cr.x)) * (float)kHalfLog2e;
    if (mixed) {
      float sg = fmaf(v, r.p4.w, fmaf(u, r.p3.w, r.p5.w));
      sg = fmaf(dt, fmaf(v, r.p9.w, fmaf(u, r.p8.w, r.p7.w)), sg);
      reject(!(sg < 0.0f || !__builtin_signbitf(r.flag)), o);
    }
    o->dg = dg;
    o->cr = cr;
  }
}
template <bool RS>
__device__ __forceinline__ bool eval_hit(const PairRegs<RS>& r, const Eval& o) {
  return o.cc <= r.Kp * o.dd;
}

// Stage 2 (only for waves where some pixel passed): alpha = min(sigma rho, alpha_max)
// with sigma rho = 2^(lsig - omega'^2), or for a degree-n response (GEN)
// 2^(lsig - x), x = 2^(k_h log2 omega'^2 + k_l).
template <bool RS, bool GEN>
__device__ __forceinline__ void eval_alpha(const PairRegs<RS>& r, const Thresholds& th, Eval* o) {
  const float amax = th.alpha_max;
  const float idd = __builtin_amdgcn_rcpf(o->dd);
  float araw;
  if (GEN) {
    o->lq = __builtin_amdgcn_logf(o->cc * idd);  // log2; -inf at the centre line
    araw = __builtin_amdgcn_exp2f(r.lsig - __builtin_amdgcn_exp2f(fmaf(th.k_h, o->lq, th.k_l)));
  } else {
    araw = __builtin_amdgcn_exp2f(fmaf(-o->cc, idd, r.lsig));
  }
  o->idd = idd;
  o->araw = araw;
  o->clamped = araw > amax;
  // araw >= 0, so med3(araw, 0, amax) = min(araw, amax) in one instruction;
  // callers use a only where eval_hit holds
  o->a = __builtin_amdgcn_fmed3f(araw, 0.0f, amax);
}

// Hybrid rendering (Sec. 6.2): does the pair's maximum-response point lie
// beyond the pixel's clip distance (its closest surface intersection)?  With
// d = n + u e1 + v e2 (|d| = dlen = sqrt(1 + u^2 + v^2)) the hit is at
// tau' = -(o_g . d_g) / |d_g|^2 along d, i.e. at distance tau' dlen, so it is
// behind when -(o_g . d_g) dlen > clip |d_g|^2.  o_g . d_g is the same affine
// (bilinear under a rolling shutter) form as the tau_max sign test.  Forward
// and backward call this with the same operands.
template <bool RS>
__device__ __forceinline__ void clip_test(const PairRegs<RS>& r, const float4* P, float u, float v,
                                          float dt, float dlen, float clip, Eval* o) {
  float odg;
  if (!RS) {
    const float4 p5 = P[5];
    odg = fmaf(v, p5.z, fmaf(u, p5.y, p5.x));
  } else {
    odg = fmaf(v, r.p4.w, fmaf(u, r.p3.w, r.p5.w));
    odg = fmaf(dt, fmaf(v, r.p9.w, fmaf(u, r.p8.w, r.p7.w)), odg);
  }
  reject(-odg * dlen > clip * o->dd, o);
}

// Colour of a pair (FP64 slots).
template <bool RS>
__device__ __forceinline__ void pair_colour(const float4* P, double c[3]) {
  const double2 rg = reinterpret_cast<const double2*>(P + (RS ? 6 : 4))[0];
  c[0] = rg.x;
  c[1] = rg.y;
  c[2] = reinterpret_cast<const double*>(P + (RS ? 10 : 6))[0];
}

// Backward only: d_g and o_g x d_g on the pixel ray (unscaled), for the
// closest point p = d_g x (o_g x d_g) / |d_g|^2.
template <bool RS>
__device__ __forceinline__ void pair_vectors(const float4* P, const Eval& ev, float u, float v,
                                             float3* dg, float3* cr) {
  if (RS) {
    *dg = ev.dg;
    *cr = ev.cr;
  } else {
    const float4 q6 = P[7], q7 = P[8], q8 = P[9], q9 = P[10], q10 = P[11];
    *dg = f3(fmaf(v, q8.x, fmaf(u, q7.x, q6.x)), fmaf(v, q8.y, fmaf(u, q7.y, q6.y)),
             fmaf(v, q8.z, fmaf(u, q7.z, q6.z)));
    *cr = f3(fmaf(v, q9.w, fmaf(u, q9.x, q6.w)), fmaf(v, q10.x, fmaf(u, q9.y, q7.w)),
             fmaf(v, q10.y, fmaf(u, q9.z, q8.w)));
  }
}

// ---- a wave's quadrant, its four 4 x 4 blocks and their lists of pairs
//
// A tile is four 8 x 8 quadrants, each walked by one wave, and a wave is four
// rows of 16 lanes, one 4 x 4 pixel block each.  A row walks its own list of
// pairs, so one step of a wave takes up to four different pairs, one per
// block, and a pair costs a step only for the blocks it can reach.  The
// particles are a few pixels wide: of the 8 x 8 quadrants that a pair reaches,
// half the 4 x 4 blocks are missed (1M particles, 1920x1080: 3.27M quadrants
// against 10.2M blocks, 2.5M steps, pinhole; 2.35M against 5.4M, 1.35M steps,
// fisheye; 300k, 800x600 rolling: 0.52M against 0.90M, 0.22M steps).
__device__ inline void lane_pixel(int q, int lane, int* x, int* y) {  // of quadrant q
  *x = 8 * (q & 1) + 4 * ((lane >> 4) & 1) + (lane & 3);
  *y = 8 * (q >> 1) + 4 * (lane >> 5) + ((lane >> 2) & 3);
}

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or_self(float x) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, ROWS, 0xF, false));
}
// (med3 against an infinity: a max or min that does not quieten its operands first)
struct OpMax {
  __device__ float operator()(float a, float b) const { return __builtin_amdgcn_fmed3f(a, b, INFINITY); }
};
struct OpMin {
  __device__ float operator()(float a, float b) const { return __builtin_amdgcn_fmed3f(a, b, -INFINITY); }
};
// Reduction over each row of 16 lanes, in all its lanes (DPP rotations: two
// instructions a step, where a shuffle through LDS takes about six).
template <class Op>
__device__ __forceinline__ float row_reduce(float x) {
  Op op;
  x = op(x, dpp_or_self<0x128, 0xF>(x));
  x = op(x, dpp_or_self<0x124, 0xF>(x));
  x = op(x, dpp_or_self<0x122, 0xF>(x));
  return op(x, dpp_or_self<0x121, 0xF>(x));
}
// From there over the wave's four rows, in lane 63 (row broadcasts).
template <class Op>
__device__ __forceinline__ float rows_reduce63(float x) {
  Op op;
  x = op(x, dpp_or_self<0x142, 0xA>(x));
  return op(x, dpp_or_self<0x143, 0xC>(x));
}

// Block-wide maxima of |u|, |v|, |dt| over the tile's valid pixels (NQ per
// thread, in a block of 256 / NQ).
template <int NQ>
__device__ inline void tile_bounds(const float* u, const float* v, const float* dt, const bool* valid,
                                   float* red, float* umax, float* vmax, float* dtmax) {
  float a = 0.0f, b = 0.0f, c = 0.0f;
#pragma unroll
  for (int k = 0; k < NQ; k++) {
    a = valid[k] ? fmaxf(a, fabsf(u[k])) : a;
    b = valid[k] ? fmaxf(b, fabsf(v[k])) : b;
    c = valid[k] ? fmaxf(c, fabsf(dt[k])) : c;
  }
  a = rows_reduce63<OpMax>(row_reduce<OpMax>(a));
  b = rows_reduce63<OpMax>(row_reduce<OpMax>(b));
  c = rows_reduce63<OpMax>(row_reduce<OpMax>(c));
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) { red[3 * w] = a; red[3 * w + 1] = b; red[3 * w + 2] = c; }
  __syncthreads();
  float A = 0, B = 0, Cc = 0;
#pragma unroll
  for (int k = 0; k < 4 / NQ; k++) {
    A = fmaxf(A, red[3 * k]);
    B = fmaxf(B, red[3 * k + 1]);
    Cc = fmaxf(Cc, red[3 * k + 2]);
  }
  // a little slack so the FP64 sign classification covers FP32 rounding of u, v
  *umax = A * 1.0001f + 1e-7f;
  *vmax = B * 1.0001f + 1e-7f;
  *dtmax = Cc * 1.0001f + 1e-7f;
}

// Pixel box of the lane's 4 x 4 block, a little larger than the pixels (by
// more than FP32 rounding of an ellipse's centre within the tile).
struct BlockBox {
  float u0, u1, v0, v1;
};
// The lane's block box; the box of the wave's quadrant k goes to LDS.
__device__ inline BlockBox block_box(float u, float v, bool valid, float slack, int k, QuadBoxes* wb) {
  BlockBox b;
  b.u0 = row_reduce<OpMin>(valid ? u : 3e38f);
  b.u1 = row_reduce<OpMax>(valid ? u : -3e38f);
  b.v0 = row_reduce<OpMin>(valid ? v : 3e38f);
  b.v1 = row_reduce<OpMax>(valid ? v : -3e38f);
  const float a0 = rows_reduce63<OpMin>(b.u0), a1 = rows_reduce63<OpMax>(b.u1);
  const float b0 = rows_reduce63<OpMin>(b.v0), b1 = rows_reduce63<OpMax>(b.v1);
  if ((threadIdx.x & 63) == 63) {
    wb->u0[k] = a0; wb->u1[k] = a1; wb->v0[k] = b0; wb->v1[k] = b1;
  }
  b.u0 -= slack; b.u1 += slack; b.v0 -= slack; b.v1 += slack;
  return b;
}

// Largest clip distance over quadrant k's valid pixels (+inf if any is
// unclipped; -inf if the quadrant has no valid pixel).
__device__ inline void quad_clip_max(float clip, bool valid, int k, QuadBoxes* wb) {
  const float c = rows_reduce63<OpMax>(row_reduce<OpMax>(valid ? clip : -INFINITY));
  if ((threadIdx.x & 63) == 63) wb->cmax[k] = c;
}

// A batch's pairs lie in LDS in chunks of kChunk rows, each followed by a row
// for a pair that hits nothing (kChunk as a place in the chunk).
constexpr int kChunk = 128;
__host__ __device__ constexpr int batch_rows(int batch) { return batch + (batch + kChunk - 1) / kChunk; }
__device__ __forceinline__ int batch_row(int t) { return t + t / kChunk; }
// Slot t of that row: omega^2 = 0, |d_g| = 1, Kp = -1.
template <bool RS>
__device__ __forceinline__ float4 dummy_slot(int t) {
  return RS ? make_float4(t == 0 ? 1.0f : 0.0f, 0.0f, 0.0f, t == 2 ? -1.0f : 0.0f)
            : make_float4(0.0f, 0.0f, t == 3 ? 1.0f : 0.0f, t == 0 ? -1.0f : 0.0f);
}
// The rows behind each chunk (forward).
template <bool RS>
__device__ inline void write_dummies(float4* pd, int batch) {
  constexpr int S = Slots<RS, false>::N;
  const int t = threadIdx.x;
  if (t >= S) return;
  const float4 d = dummy_slot<RS>(t);
  for (int c = 1; c <= (batch + kChunk - 1) / kChunk; c++) pd[(c * (kChunk + 1) - 1) * S + t] = d;
}

// A wave's lists: of each of its blocks, the places in the chunk of the pairs
// that may reach it, in order, padded to the longest and by four more with
// kChunk.
constexpr int kListStride = kChunk + 4;
struct WaveLists {
  unsigned char row[4][kListStride];
  unsigned char quad[kChunk];  // the pairs that reach the quadrant
};

// Builds the wave's lists for one chunk (pd: its first row, pf: its pairs'
// flags) of quadrant q and returns the longest's length, with kMixed set if
// the sign of o_g . d_g varies over the tile for one of their pairs.  The
// pairs flagged for quadrant q are packed first; then each row of lanes tests 16 of them at a time against
// its own block (a convex quadratic over a box as in ellipse_meets_box, here
// in FP32 with slack for its rounding, relative to the quadratic's own terms
// and 1e-4 of the ellipse, whose K' already carries 1e-3), so the test costs
// about three instructions per pair and quadrant.  run: the lane's pixel has
// not stopped; a block without such a pixel takes no pairs.
constexpr uint32_t kMixed = 1u << 31;
template <bool RS, bool BWD>
__device__ inline uint32_t build_lists(const float4* pd, const unsigned short* pf, int q, const BlockBox& box,
                                       bool run, WaveLists& L) {
  constexpr int S = Slots<RS, BWD>::N;
  const int lane = threadIdx.x & 63, j0 = lane & 15;
  const uint32_t f0 = pf[lane], f1 = pf[lane + 64];
  const unsigned long long m0 = __builtin_amdgcn_ballot_w64((f0 >> q & 1u) != 0u);
  const unsigned long long m1 = __builtin_amdgcn_ballot_w64((f1 >> q & 1u) != 0u);
  const int c0 = __builtin_popcountll(m0), F = c0 + __builtin_popcountll(m1);
  if (F == 0) return 0u;
  const unsigned long long x0 = __builtin_amdgcn_ballot_w64((f0 & kMixedBit) != 0u);
  const unsigned long long x1 = __builtin_amdgcn_ballot_w64((f1 & kMixedBit) != 0u);
  const uint32_t mixed = ((m0 & x0) | (m1 & x1)) != 0ull ? kMixed : 0u;
  auto below = [](unsigned long long m) __attribute__((always_inline)) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  };
  if (f0 >> q & 1u) L.quad[below(m0)] = (unsigned char)lane;
  if (f1 >> q & 1u) L.quad[c0 + below(m1)] = (unsigned char)(lane + 64);
  __builtin_amdgcn_wave_barrier();  // (one wave's LDS accesses stay in order)
  auto row_bits = [&](unsigned long long m) __attribute__((always_inline)) {
    return (lane & 32 ? (uint32_t)(m >> 32) : (uint32_t)m) >> (lane & 16) & 0xffffu;
  };
  const bool alive = row_bits(__builtin_amdgcn_ballot_w64(run)) != 0u;
  unsigned char* mine = L.row[lane >> 4];
  uint32_t cnt = 0;
  for (int it = 0; it < F; it += 16) {
    const int j = it + j0;
    const uint32_t i = L.quad[min(j, F - 1)];
    const float4* P = pd + i * S;
    const float2 c = reinterpret_cast<const float2*>(P + (RS ? 10 : 6))[1];
    const float E11 = fabsf(P[RS ? 0 : 2].w), E12 = RS ? P[11].x : P[3].w, E22 = RS ? P[11].y : P[5].w;
    const float a0 = box.u0 - c.x, a1 = box.u1 - c.x, b0 = box.v0 - c.y, b1 = box.v1 - c.y;
    const float x = __builtin_amdgcn_fmed3f(0.0f, a0, a1), y = __builtin_amdgcn_fmed3f(0.0f, b0, b1);
    const float ye = __builtin_amdgcn_fmed3f(-E12 * x * __builtin_amdgcn_rcpf(E22), b0, b1);
    const float xe = __builtin_amdgcn_fmed3f(-E12 * y * __builtin_amdgcn_rcpf(E11), a0, a1);
    auto meets = [&](float X, float Y) __attribute__((always_inline)) {
      const float d = fmaf(E11 * X, X, E22 * Y * Y);
      return !(fmaf(2.0f * E12 * X, Y, d) > fmaf(4e-6f, d, 1.0001f));  // (a NaN counts as a hit)
    };
    const bool keep = j < F && alive && (meets(x, ye) || meets(xe, y));
    const uint32_t bits = row_bits(__builtin_amdgcn_ballot_w64(keep));
    if (keep) mine[cnt + __builtin_popcount(bits & ((1u << j0) - 1u))] = (unsigned char)i;
    cnt += __builtin_popcount(bits);
  }
  const uint32_t n0 = __builtin_amdgcn_readlane(cnt, 0), n1 = __builtin_amdgcn_readlane(cnt, 16);
  const uint32_t n2 = __builtin_amdgcn_readlane(cnt, 32), n3 = __builtin_amdgcn_readlane(cnt, 48);
  const uint32_t most = max(max(n0, n1), max(n2, n3));
  for (uint32_t k = cnt + j0; k < most + 4; k += 16) mine[k] = (unsigned char)kChunk;
  __builtin_amdgcn_wave_barrier();
  return __builtin_amdgcn_readfirstlane(most | mixed);
}

// True when pred holds on some active lane (the wave's lane mask, without a
// round trip through a vector register).
__device__ __forceinline__ bool wave_any(bool pred) {
  return __builtin_amdgcn_ballot_w64(pred) != 0ull;
}

}  // namespace gut
