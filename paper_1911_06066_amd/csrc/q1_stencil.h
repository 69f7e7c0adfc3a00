// Matrix-free Q1 operators on structured grids (node-centred gather).
//
// For an axis-aligned box element with sides (hx, hy[, hz]) and a constant
// tensor D, the element mass and stiffness matrices are tensor products of the
// 1D matrices  m = h/6 [2 1; 1 2],  k = 1/h [1 -1; -1 1],  g = int phi_a' phi_b = s_a / 2
// (s_0 = -1, s_1 = +1).  Contracting them with the element's vertex values in
// closed form gives the row of node v of  M_e mv + K_e kv  with a few dozen
// flops; a node sums the rows of its 4 (2D) or 8 (3D) adjacent elements.  The
// result is y = M mv + K kv for two nodal fields mv, kv -- the Jacobian slab
// operator uses mv = (1/dt - f'(u)) x, kv = x; the residual uses
// mv = (u_k - u_{k-1})/dt - f(u_k), kv = u_k.
//
// Field accessors take node coordinates (ii, jj[, kk]), already clamped to the
// grid, so the same code reads global memory or an LDS tile.
#pragma once

#include "stm_device.h"

namespace stm {

template <typename T>
struct Tensor2 { T xx, yy, xy; };

template <typename T>
struct Tensor3 { T xx, yy, zz, xy; };  // fibres lie in the x-y plane: xz = yz = 0

// y for node (i, j).  fm(ii, jj), fk(ii, jj): nodal values; fd(ex, ey): Tensor2.
// diag (optional): diagonal of  M diag(w) + K  at the node, w = wself there.
template <typename T, typename FM, typename FK, typename FD>
__device__ __forceinline__ T q1_apply_2d(const GridDev& g, int i, int j, FM fm, FK fk, FD fd, T wself, T* diag) {
  T mv[3][3], kv[3][3];
#pragma unroll
  for (int dj = 0; dj < 3; ++dj) {
    const int jj = min(max(j + dj - 1, 0), g.ny - 1);
#pragma unroll
    for (int di = 0; di < 3; ++di) {
      const int ii = min(max(i + di - 1, 0), g.nx - 1);
      mv[dj][di] = fm(ii, jj);
      kv[dj][di] = fk(ii, jj);
    }
  }
  const T cxx = T(g.hy / (6.0 * g.hx));
  const T cyy = T(g.hx / (6.0 * g.hy));
  const T cm = T(g.hx * g.hy / 36.0);
  T y = T(0), dg = T(0);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int ey = j - 1 + b;
    if (ey < 0 || ey >= g.ey) continue;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int ex = i - 1 + a;
      if (ex < 0 || ex >= g.ex) continue;
      const Tensor2<T> D = fd(ex, ey);
      const T sx = T(1 - 2 * a), sy = T(1 - 2 * b);
      // differences along x on the node's row and the opposite row
      const T dxv = kv[1][a + 1] - kv[1][a];
      const T dxo = kv[2 * b][a + 1] - kv[2 * b][a];
      // differences along y on the node's column and the opposite column
      const T dyv = kv[b + 1][1] - kv[b][1];
      const T dyo = kv[b + 1][2 * a] - kv[b][2 * a];
      T acc = cxx * D.xx * sx * (T(2) * dxv + dxo);
      acc += cyy * D.yy * sy * (T(2) * dyv + dyo);
      acc += T(0.25) * D.xy * (sx * (dyv + dyo) + sy * (dxv + dxo));
      acc += cm * (T(4) * mv[1][1] + T(2) * mv[1][2 * a] + T(2) * mv[2 * b][1] + mv[2 * b][2 * a]);
      y += acc;
      if (diag) dg += T(2) * cxx * D.xx + T(2) * cyy * D.yy + T(0.5) * D.xy * sx * sy + T(4) * cm * wself;
    }
  }
  if (diag) *diag = dg;
  return y;
}

// 3D: node (i, j, k).  Element vertex (wx, wy, wz) of the element at offset
// (a, b, c) (ex = i-1+a ...) sits at stencil position (a+wx, b+wy, c+wz).
// The 1D factors along each axis: mass m(v,w) = h/6 (2 if v==w else 1),
// stiffness k(v,w) = s_v s_w / h, mixed g(v,w) = s_v / 2.
template <typename T, typename FM, typename FK, typename FD>
__device__ __forceinline__ T q1_apply_3d(const GridDev& g, int i, int j, int k, FM fm, FK fk, FD fd, T wself,
                                         T* diag) {
  T mv[3][3][3], kv[3][3][3];
#pragma unroll
  for (int dk = 0; dk < 3; ++dk) {
    const int kk = min(max(k + dk - 1, 0), g.nz - 1);
#pragma unroll
    for (int dj = 0; dj < 3; ++dj) {
      const int jj = min(max(j + dj - 1, 0), g.ny - 1);
#pragma unroll
      for (int di = 0; di < 3; ++di) {
        const int ii = min(max(i + di - 1, 0), g.nx - 1);
        mv[dk][dj][di] = fm(ii, jj, kk);
        kv[dk][dj][di] = fk(ii, jj, kk);
      }
    }
  }
  const T hx = T(g.hx), hy = T(g.hy), hz = T(g.hz);
  const T cxx = hy * hz / (T(36) * hx), cyy = hx * hz / (T(36) * hy), czz = hx * hy / (T(36) * hz);
  const T cxy = hz / T(24), cm = hx * hy * hz / T(216);
  T y = T(0), dg = T(0);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int ez = k - 1 + c;
    if (ez < 0 || ez >= g.ez) continue;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int ey = j - 1 + b;
      if (ey < 0 || ey >= g.ey) continue;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int ex = i - 1 + a;
        if (ex < 0 || ex >= g.ex) continue;
        const Tensor3<T> D = fd(ex, ey, ez);
        // local vertex of the node: (1-a, 1-b, 1-c); signs s = 2v - 1
        const T sx = T(1 - 2 * a), sy = T(1 - 2 * b), sz = T(1 - 2 * c);
        // Sum over the 8 element vertices w of  A_vw x_w  with
        //   xx: (sx sw_x / hx) (hy/6 my) (hz/6 mz),  likewise yy, zz
        //   xy + yx: (sx/2)(sw_y/2)(hz/6 mz) + (sw_x/2)(sy/2)(hz/6 mz)
        //   mass: (hx/6 mx)(hy/6 my)(hz/6 mz)
        T sxx = T(0), syy = T(0), szz = T(0), sxy = T(0), smm = T(0);
#pragma unroll
        for (int wz = 0; wz < 2; ++wz) {
#pragma unroll
          for (int wy = 0; wy < 2; ++wy) {
#pragma unroll
            for (int wx = 0; wx < 2; ++wx) {
              const T xk = kv[c + wz][b + wy][a + wx];
              const T xm = mv[c + wz][b + wy][a + wx];
              const T mx = (wx == 1 - a) ? T(2) : T(1);
              const T my = (wy == 1 - b) ? T(2) : T(1);
              const T mz = (wz == 1 - c) ? T(2) : T(1);
              const T swx = T(2 * wx - 1), swy = T(2 * wy - 1), swz = T(2 * wz - 1);
              sxx += swx * my * mz * xk;
              syy += swy * mx * mz * xk;
              szz += swz * mx * my * xk;
              sxy += (sx * swy + swx * sy) * mz * xk;
              smm += mx * my * mz * xm;
            }
          }
        }
        T acc = D.xx * sx * sxx * cxx;
        acc += D.yy * sy * syy * cyy;
        acc += D.zz * sz * szz * czz;
        acc += D.xy * sxy * cxy;
        acc += smm * cm;
        y += acc;
        if (diag) {
          dg += T(4) * (D.xx * cxx + D.yy * cyy + D.zz * czz) + T(4) * D.xy * sx * sy * cxy +
                T(8) * cm * wself;
        }
      }
    }
  }
  if (diag) *diag = dg;
  return y;
}

}  // namespace stm

namespace stm {

// ---------------------------------------------------------------------------
// Element-centred evaluation: the contributions of one element to its
// vertices, out[v] = (M_e m + K_e k)_v, with the 1D factors applied axis by
// axis (sum factorisation).  Vertex v = bx + 2 by (+ 4 bz).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void elem_apply_2d(const T (&k)[4], const T (&m)[4], const Tensor2<T>& D, T cxx, T cyy,
                                              T cm, T (&out)[4]) {
  const T dx0 = k[1] - k[0], dx1 = k[3] - k[2];
  const T dy0 = k[2] - k[0], dy1 = k[3] - k[1];
  const T p0 = cxx * D.xx * (T(2) * dx0 + dx1), p1 = cxx * D.xx * (T(2) * dx1 + dx0);
  const T q0 = cyy * D.yy * (T(2) * dy0 + dy1), q1 = cyy * D.yy * (T(2) * dy1 + dy0);
  const T A = T(0.25) * D.xy * (dy0 + dy1), B = T(0.25) * D.xy * (dx0 + dx1);
  const T r00 = T(2) * m[0] + m[1], r01 = m[0] + T(2) * m[1];  // row by=0: vx = 0, 1
  const T r10 = T(2) * m[2] + m[3], r11 = m[2] + T(2) * m[3];  // row by=1
  out[0] = -p0 - q0 - A - B + cm * (T(2) * r00 + r10);
  out[1] = p0 - q1 + A - B + cm * (T(2) * r01 + r11);
  out[2] = -p1 + q0 - A + B + cm * (T(2) * r10 + r00);
  out[3] = p1 + q1 + A + B + cm * (T(2) * r11 + r01);
}

// The 3D element in the basis of sums and differences: per axis a vertex pair
// (v0, v1) becomes s = v0 + v1, d = v1 - v0.  There the 1D mass factor
// [[2, 1], [1, 2]] is diag(3, 1), the stiffness factor [[1, -1], [-1, 1]] is
// diag(0, 2), and the mixed one takes s to d.  With m(abc) = 3^(number of s)
// over the three axes and ax = D_xx h_y h_z / (36 h_x), ay, az likewise,
// axy = D_xy h_z / 24 and cm = h_x h_y h_z / 216 (a constant tensor whose fibres
// lie in the x-y plane), K_e k + M_e mv is
//   d..: 2 ax m / 3^[..] k(d..) + 4 axy 3^[z = s] k(sd.) (for ds.), y and z likewise,
//   plus cm m mv,
// and the way back to the vertices takes 1/2 per axis.  An x-y face is
// transformed once for the two layers it bounds; a layer needs the sums and
// differences of its two faces, 11 products for the stiffness and 8 for the mass.
template <typename T>
__device__ __forceinline__ void face_transform(const T (&v)[4], T (&h)[4]) {
  const T s0 = v[0] + v[1], d0 = v[1] - v[0], s1 = v[2] + v[3], d1 = v[3] - v[2];
  h[0] = s0 + s1;  // ss
  h[1] = d0 + d1;  // ds
  h[2] = s1 - s0;  // sd
  h[3] = d1 - d0;  // dd
}

// One element layer between its bottom face (kb, mb) and top face (kt, mt), all
// transformed in x and y.  gx = 3/4 ax (gy, gz likewise), gxy = axy / 2,
// c1 = cm / 8, c3 = 3 c1, c9 = 9 c1.  bottom: carry plus the layer's
// contribution to the lower plane; carry: its contribution to the upper plane.
template <typename T>
__device__ __forceinline__ void layer_apply(const T (&kb)[4], const T (&kt)[4], const T (&mb)[4], const T (&mt)[4],
                                            T gx, T gy, T gz, T gxy, T c1, T c3, T c9, T (&carry)[4],
                                            T (&bottom)[4]) {
  const T k1s = kb[1] + kt[1], k2s = kb[2] + kt[2], k3s = kb[3] + kt[3];
  const T k0d = kt[0] - kb[0], k1d = kt[1] - kb[1], k2d = kt[2] - kb[2], k3d = kt[3] - kb[3];
  const T third = T(1) / T(3);
  const T gxz = gx + gz, gyz = gy + gz, gs = gx + gy;
  // a third of the z-sum's part, and the z-difference's part
  const T s0 = c9 * (mb[0] + mt[0]);
  const T s1 = fma(gx, k1s, fma(gxy, k2s, c3 * (mb[1] + mt[1])));
  const T s2 = fma(gy, k2s, fma(gxy, k1s, c3 * (mb[2] + mt[2])));
  const T s3 = fma(gs * third, k3s, c1 * (mb[3] + mt[3]));
  const T d0 = fma(T(3) * gz, k0d, c9 * (mt[0] - mb[0]));
  const T d1 = fma(gxz, k1d, fma(gxy, k2d, c3 * (mt[1] - mb[1])));
  const T d2 = fma(gyz, k2d, fma(gxy, k1d, c3 * (mt[2] - mb[2])));
  const T d3 = fma((gs + gz) * third, k3d, c1 * (mt[3] - mb[3]));
  bottom[0] = fma(T(3), s0, carry[0]) - d0;
  bottom[1] = fma(T(3), s1, carry[1]) - d1;
  bottom[2] = fma(T(3), s2, carry[2]) - d2;
  bottom[3] = fma(T(3), s3, carry[3]) - d3;
  carry[0] = fma(T(3), s0, d0);
  carry[1] = fma(T(3), s1, d1);
  carry[2] = fma(T(3), s2, d2);
  carry[3] = fma(T(3), s3, d3);
}

}  // namespace stm
