// WENO5 stage kernel (Sec. 3.2 limiter list: the fifth-order WENO
// reconstruction of Jiang and Shu, three ghost layers).
//
// One workgroup per tile of TS x TS columns of a block (8 x 8 for 8^d blocks,
// 16 x 16 for 16^d and 32^d), thread (i, j) owning column (i, j) and marching
// it in z (a 2-D tile is one plane).  Per plane the primitives of the tile and
// of its three-deep x and y halos are staged in LDS; every thread reconstructs
// its own cell along x, y and z, both face values at once, and then evaluates
// the flux through its lower x and y face and its upper z face.  Halo cells
// across a same-level face are read straight from the neighbouring block when
// the mesh gathers halos, else (and always across refinement and boundary
// faces) from the block's stored ghosts.  The update, the refinement-face flux
// capture, the gravity source and the CFL epilogue follow the plane-marching
// stage kernel: stage 1 / 2 Heun's stages, 3 the generic sub-step, 4 the
// generic sub-step with three earlier states.
//
// Bound by VALU issue: the reconstruction.  Per cell, not per face, because
// the smoothness indicators of a cell's three stencils serve both of its face
// values (the mirrored stencil has the same indicators in reverse order): per
// variable and axis about 65 issue slots for both values, against twice 67
// when each side of each face is reconstructed for itself.  Face values and
// fluxes share one LDS slot per face (26.9 kB FP32 for a 16 x 16 tile), and the
// loads of the next plane are issued after the reconstructions, which leaves
// FP32 16 x 16 tiles at 114-127 registers, four waves per SIMD, no spills.
// 160 x 160 x 192 cells in 16^3 blocks, FP32, walls and gravity, two Heun steps:
// 1840 us with per-face reconstruction and stored ghosts (1510 us of it in the
// stages), 765 us now; 768^2 cells in 32^2 blocks, FP64, HLL, two SSP-RK3 steps:
// 397 us with every face evaluated by both of its cells, 184 us now.
#include "device_common.h"
#include "foap4_internal.h"
#include "stage_common.h"

namespace f4 {

// FP32: the squared reciprocals of three positive values; FP64: the same
// weights times the product of the three squares (their ratios are all that
// counts), which needs no reciprocal.  With the differences that they multiply
// the products stay finite for values below about 1e68, which are differences
// of neighbouring cells of about 1e34.
__device__ __forceinline__ void weno_weights(const float *b, float *R) {
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const float r = frcp(b[k]);
    R[k] = r * r;
  }
}
__device__ __forceinline__ void weno_weights(const double *b, double *R) {
  const double E0 = b[0] * b[0], E1 = b[1] * b[1], E2 = b[2] * b[2];
  R[0] = E1 * E2;
  R[1] = E0 * E2;
  R[2] = E0 * E1;
}

// Values of cell v2 at its lower (lo) and upper (hi) face from v0 .. v4: the
// convex combinations of the third-order candidates with the weights
// alpha_k / sum alpha, alpha_k = d_k / (eps + beta_k)^2, eps = 1e-6,
// d = (1, 6, 3)/10 at the upper face and reversed at the lower one, beta_k the
// candidates' smoothness indicators 13/12 s^2 + 1/4 t^2.  Written in the
// differences of neighbouring cells, with all (eps + beta_k) scaled by 12/13:
// each candidate is v2 plus q_k / 6.
template <typename T>
__device__ __forceinline__ void weno5(T v0, T v1, T v2, T v3, T v4, T &lo, T &hi) {
  const T d1 = v1 - v0, d2 = v2 - v1, d3 = v3 - v2, d4 = v4 - v3;
  const T s0 = d2 - d1, s1 = d3 - d2, s2 = d4 - d3;
  const T t0 = T(3) * d2 - d1, t1 = d2 + d3, t2 = d4 - T(3) * d3;
  const T c = T(3.0 / 13.0), e = T(12e-6 / 13.0);
  const T b[3] = {(c * t0) * t0 + (s0 * s0 + e), (c * t1) * t1 + (s1 * s1 + e), (c * t2) * t2 + (s2 * s2 + e)};
  T R[3];
  weno_weights(b, R);
  const T m = T(6) * R[1], h2 = T(3) * R[2], l0 = T(3) * R[0];
  const T sh = (R[0] + m) + h2, sl = (R[2] + m) + l0;
  const T qh = R[0] * (T(2) * t0 - d2) + m * (T(2) * d3 + d2) + h2 * (d3 - t2);
  const T ql = R[2] * (T(2) * t2 + d3) - m * (T(2) * d2 + d3) - l0 * (d2 + t0);
  hi = v2 + T(1.0 / 6.0) * (qh * frcp(sh));
  lo = v2 + T(1.0 / 6.0) * (ql * frcp(sl));
}

// Keeps the reconstructions of a cell's variables and axes in source order:
// interleaved, as the compiler would schedule them, they hold three times the
// registers and spill.
template <typename T>
__device__ __forceinline__ void pin(T &a, T &b) {
  asm volatile("" : "+v"(a), "+v"(b)::"memory");
}
template <typename T>
__device__ __forceinline__ void pin(T &a) {
  asm volatile("" : "+v"(a)::"memory");
}

// Tile shape of a block size, and LDS layout.  FP32 rows of the staged plane are
// LP = 24 values apart: 24 = -8 mod 32 banks, so the half waves of an 8 x 8
// tile (four adjacent rows) and of a 16 x 16 tile (rows r and r + 2, see the
// lane map) touch every bank once.  FP64 rows are tight (TS + 6 and TS + 1
// values), so that four 2D workgroups share a CU (34 kB each; 43 kB at 24 values
// a row, three): 194 -> 182 us for the 2D case above.
template <typename T, int TS>
struct WenoTile {
  static constexpr int Q = TS + 6;                           // plane rows -3 .. TS + 2
  static constexpr int LP = sizeof(T) == 4 ? 24 : Q;         // their stride
  static constexpr int PLANE = Q * LP;
  static constexpr int LF = sizeof(T) == 4 ? 24 : TS + 1;    // row stride of the face values
  static constexpr int FACES = (TS + 1) * LF;
  static constexpr int RING = (12 * TS + TS * TS - 1) / (TS * TS);  // halo cells per thread
};

template <typename T, int NDIM, int TS, int SCH, int STG>
__global__ __launch_bounds__(TS *TS) void weno_kernel(const MeshDev *__restrict__ Mp, int64_t total, int kd, SubStep ss) {
  using C = WenoTile<T, TS>;
  constexpr int NV = NDIM + 2, NF = 2 * NDIM, LP = C::LP, LF = C::LF, PLANE = C::PLANE, RING = C::RING;
  __shared__ T Ws[NV * PLANE];     // primitives: cell (x, y) at (y + 3) LP + x + 3
  __shared__ T Fx[NV * C::FACES];  // face x - 1/2 of row y at y LF + x: left value, then flux
  __shared__ T Fy[NV * C::FACES];  // face y - 1/2 of column x at y LF + x
  const MeshDev &M = *Mp;
  // XCD-aware tile order: XCD x = w mod 8 takes the contiguous tiles
  // [x q + min(x, r), ...), total = 8 q + r
  const int64_t xq = total / 8, xr = total % 8, xid = blockIdx.x % 8;
  const int64_t item = xid * xq + (xid < xr ? xid : xr) + blockIdx.x / 8;
  const int N = M.N, g = M.g, P = N + 2 * g, tpr = N / TS, tpb = tpr * tpr;
  const int slabs = NDIM == 3 ? N / kd : 1;  // slabs of kd planes per tile
  const int64_t col = item / slabs, b = col / tpb;
  const int k0 = NDIM == 3 ? (int)(item % slabs) * kd : 0, k1 = NDIM == 3 ? k0 + kd : 1;
  const int tile = (int)(col % tpb), i0 = (tile % tpr) * TS, j0 = (tile / tpr) * TS;
  const int t = threadIdx.x;
  int ti, tj;
  if constexpr (TS == 16) {  // wave w: rows 8 (w / 2) + (w & 1) + {0, 2, 4, 6}
    const int w = t >> 6, l = t & 63;
    ti = l & 15;
    tj = 8 * (w >> 1) + (w & 1) + 2 * (l >> 4);
  } else {
    ti = t & 7;
    tj = t >> 3;
  }
  const int I = i0 + ti, J = j0 + tj;
  const int sk = P * N;
  const int sv = (NDIM == 3) ? P * P * P : P * P;
  const int64_t bel = (int64_t)sv * NV;
  const int cur = M.cur;
  const T *ud0 = (const T *)M.s[STG >= 3 ? role_buffer(ss.deriv, cur) : (STG == 1 ? cur : 1 - cur)];
  const T *ud = ud0 + b * bel;
  T *uo = (T *)M.s[STG >= 3 ? role_buffer(ss.out, cur) : (STG == 1 ? 1 - cur : cur)] + b * bel;
  const T *up = (const T *)M.s[STG >= 3 ? role_buffer(ss.prev, cur) : cur] + b * bel;
  const T gamma = (T)M.gamma;
  const double dx = ldexp(M.dx0, -gload(M.level + b));
  const T idx = (T)(1.0 / dx);
  const double dt = gload(M.scal + kDt);
  const T dts = (T)(STG >= 3 ? ss.c * dt : (STG == 1 ? dt : 0.5 * dt));
  const T cdt = dts * idx;
  int finfo[NF];
#pragma unroll
  for (int f = 0; f < NF; f++) finfo[f] = __builtin_amdgcn_readfirstlane(gload(M.face_info + b * NF + f));
  auto nbr = [&](int f) -> const T * {
    return (M.gather && finfo[f] <= -2) ? ud0 + (int64_t)(-2 - finfo[f]) * bel : nullptr;
  };
  // refinement-face flux F of face f at in-face position (t1, t2)
  auto bflux = [&](int f, int t1, int t2, const T *F) {
    const int info = finfo[f];
    if (info < 0) return;
    const int fv = NDIM == 3 ? N * N : N;  // values per variable
    const T *buf = (const T *)((info & 1) ? M.bflux_c : M.bflux_f) + (int64_t)(info >> 1) * (NV * fv);
    const auto r = buf_rsrc(buf);
    const uint32_t o = (uint32_t)(NDIM == 3 ? t2 * N + t1 : t1) * (uint32_t)sizeof(T);
#pragma unroll
    for (int v = 0; v < NV; v++) buf_store<T>(F[v], r, o, (uint32_t)(v * fv * (int)sizeof(T)));
  };

  // the own column: plane kk of the block (or across -z / +z of the
  // neighbour) at a wave-uniform base, plus the lane's byte offset
  const uint32_t lo_b = (uint32_t)cell_off<NDIM>(I, J, 0, N, g) * (uint32_t)sizeof(T);
  const T *zlo = nullptr, *zhi = nullptr;
  if constexpr (NDIM == 3) {
    zlo = nbr(4);
    zhi = nbr(5);
  }
  auto colb = [&](int kk) -> const T * {
    if (kk < 0 && zlo) return zlo + (kk + N) * sk;
    if (kk >= N && zhi) return zhi + (kk - N) * sk;
    return ud + kk * sk;
  };
  auto loadc = [&](const T *base, T *U) {
    const auto r = buf_rsrc(base);
#pragma unroll
    for (int v = 0; v < NV; v++) U[v] = buf_load<T>(r, lo_b, (uint32_t)(v * sv * (int)sizeof(T)));
  };
  // this thread's halo cells: strips -x, +x, -y, +y of 3 TS cells
  const T *rp[RING];
  int rs[RING], rl[RING];
#pragma unroll
  for (int q = 0; q < RING; q++) {
    const int h = t + q * TS * TS;
    rl[q] = -1;
    rp[q] = ud;
    rs[q] = 0;
    if (h >= 12 * TS) continue;
    const int strip = h / (3 * TS), r = h % (3 * TS);
    int x, y;
    if (strip < 2) {  // adjacent lanes take the three cells of a row
      y = r / 3;
      x = strip == 0 ? r % 3 - 3 : TS + r % 3;
    } else {
      x = r % TS;
      y = strip == 2 ? r / TS - 3 : TS + r / TS;
    }
    rl[q] = (y + 3) * LP + x + 3;
    x += i0;
    y += j0;
    const T *src = nullptr;
    if (x < 0) { src = nbr(0); if (src) x += N; }
    else if (x >= N) { src = nbr(1); if (src) x -= N; }
    else if (y < 0) { src = nbr(2); if (src) y += N; }
    else if (y >= N) { src = nbr(3); if (src) y -= N; }
    rp[q] = (src ? src : ud) + cell_off<NDIM>(x, y, 0, N, g);
    rs[q] = NDIM == 3 ? ((unsigned)x < (unsigned)N ? sk : P * 2 * g) : 0;
  }
  auto load_ring = [&](int kk, T (*R)[NV]) {
#pragma unroll
    for (int q = 0; q < RING; q++)
      if (rl[q] >= 0) {
#pragma unroll
        for (int v = 0; v < NV; v++) R[q][v] = gload(rp[q] + kk * rs[q] + v * sv);
      }
  };

  auto is_f2c = [&](int f) { return f < NF && finfo[f] >= 0 && (finfo[f] & 1); };
  const bool skip_xy = (is_f2c(0) && I == 0) || (is_f2c(1) && I == N - 1) || (is_f2c(2) && J == 0) ||
                       (is_f2c(3) && J == N - 1);
  const bool skip_lo = NDIM == 3 && is_f2c(4), skip_hi = NDIM == 3 && is_f2c(5);

  // z window: primitives of cells k - 1 .. k + 3 of the own column, the upper
  // face value of cell k and the flux through the lower face of plane k; the
  // conserved cell k + 4 and the next plane's halo cells are in flight
  T w[5][NV], Z[NV], Fz[NV], nx[NV], ring[RING][NV];
  T U0[NV];
  if constexpr (NDIM == 3) {
    T c6[3][NV], tmp[NV];
    loadc(colb(k0 - 3), c6[0]);
    loadc(colb(k0 - 2), c6[1]);
    loadc(colb(k0 - 1), c6[2]);
#pragma unroll
    for (int s = 0; s < 4; s++) loadc(colb(k0 + s), w[s]);
    load_ring(k0, ring);
#pragma unroll
    for (int s = 0; s < 3; s++) {
      to_prim<T, NDIM>(c6[s], gamma, tmp);
#pragma unroll
      for (int v = 0; v < NV; v++) c6[s][v] = tmp[v];
    }
#pragma unroll
    for (int s = 0; s < 4; s++) {
      to_prim<T, NDIM>(w[s], gamma, tmp);
#pragma unroll
      for (int v = 0; v < NV; v++) w[s][v] = tmp[v];
    }
    // face k0 - 1/2 from the upper value of cell k0 - 1 and the lower value of
    // cell k0; then shift the window so that it holds cells k0 - 1 .. k0 + 3
    T L[NV], R[NV], u_;
#pragma unroll
    for (int v = 0; v < NV; v++) {
      weno5(c6[0][v], c6[1][v], c6[2][v], w[0][v], w[1][v], u_, L[v]);
      pin(L[v]);
      weno5(c6[1][v], c6[2][v], w[0][v], w[1][v], w[2][v], R[v], Z[v]);
      pin(R[v], Z[v]);
    }
    riemann<T, NDIM, 2, (SCH & kSchHLL) != 0>(L, R, gamma, Fz);
    if (k0 == 0) bflux(4, I, J, Fz);
#pragma unroll
    for (int v = 0; v < NV; v++) {
      const T c3 = w[3][v];
      w[4][v] = c3;
      w[3][v] = w[2][v];
      w[2][v] = w[1][v];
      w[1][v] = w[0][v];
      w[0][v] = c6[2][v];
    }
  } else {
    load_ring(0, ring);
  }
  T vloc = T(0);
  double vmax = 0.0;
  bool bad = false;
  for (int k = k0; k < k1; k++) {
    // stage plane k
    T Up[NV];
    if constexpr (NDIM == 2) loadc(ud, U0);
    {
      T W0[NV];
      if constexpr (NDIM == 3) {
#pragma unroll
        for (int v = 0; v < NV; v++) W0[v] = w[1][v];
      } else {
        to_prim<T, NDIM>(U0, gamma, W0);
      }
#pragma unroll
      for (int v = 0; v < NV; v++) Ws[v * PLANE + (tj + 3) * LP + ti + 3] = W0[v];
#pragma unroll
      for (int q = 0; q < RING; q++)
        if (rl[q] >= 0) {
          T W[NV];
          to_prim<T, NDIM>(ring[q], gamma, W);
#pragma unroll
          for (int v = 0; v < NV; v++) Ws[v * PLANE + rl[q]] = W[v];
        }
    }
    __syncthreads();
    // x and y: the upper face value goes to the face above through LDS, the
    // lower one stays
    T xl[NV], yl[NV];
    {
      const T *c = Ws + (tj + 3) * LP + ti + 3;
#pragma unroll
      for (int v = 0; v < NV; v++, c += PLANE) {
        T hi;
        weno5(c[-2], c[-1], c[0], c[1], c[2], xl[v], hi);
        pin(xl[v], hi);
        Fx[v * C::FACES + tj * LF + ti + 1] = hi;
        weno5(c[-2 * LP], c[-LP], c[0], c[LP], c[2 * LP], yl[v], hi);
        pin(yl[v], hi);
        Fy[v * C::FACES + (tj + 1) * LF + ti] = hi;
      }
    }
    // The halo cells next to the tile: 4 TS one-sided reconstructions, one
    // wave's lanes (16 x 16 tiles: another wave each plane).  Side 0 and 2: the
    // upper value of cells -1; 1 and 3: the lower value of cells TS, whose lanes
    // also evaluate the tile's last faces.
    const int e = TS == 16 ? t - 64 * ((k + (int)item) & 3) : t;
    const bool extra = e >= 0 && e < 4 * TS;
    const int side = e / TS, em = e % TS;
    const bool ey = side >= 2, eup = side & 1;
    T E[NV];
    if (extra) {
      const int st = (ey ? LP : 1) * (eup ? -1 : 1);
      const int at = eup ? TS + 5 : 0;
      const T *c = Ws + (ey ? at * LP + em + 3 : (em + 3) * LP + at);
#pragma unroll
      for (int v = 0; v < NV; v++, c += PLANE) {
        T u_;
        weno5(c[0], c[st], c[2 * st], c[3 * st], c[4 * st], u_, E[v]);
        pin(E[v]);
      }
      if (!eup) {
        T *d = ey ? Fy + em : Fx + em * LF;
#pragma unroll
        for (int v = 0; v < NV; v++) d[v * C::FACES] = E[v];
      }
    }
    // z: cell k + 1, and the face between k and k + 1
    T Fz1[NV];
    if constexpr (NDIM == 3) {
      T R[NV], Zn[NV];
#pragma unroll
      for (int v = 0; v < NV; v++) {
        weno5(w[0][v], w[1][v], w[2][v], w[3][v], w[4][v], R[v], Zn[v]);
        pin(R[v], Zn[v]);
      }
      riemann<T, NDIM, 2, (SCH & kSchHLL) != 0>(Z, R, gamma, Fz1);
      if (k == N - 1) bflux(5, I, J, Fz1);
#pragma unroll
      for (int v = 0; v < NV; v++) Z[v] = Zn[v];
    }
    __syncthreads();
    // Loads for the update and for the next plane, issued here and not at the
    // top of the plane: in flight across the reconstructions they cost
    // registers that spill, and a reload waits for every load before it.
    if constexpr (NDIM == 3) loadc(ud + k * sk, U0);
    if constexpr (STG >= 2) loadc(up + k * sk, Up);
    if (k + 1 < k1) {
      load_ring(k + 1, ring);
      loadc(colb(k + 4), nx);
    }
    // every face's left value is read and replaced by its flux by the one
    // thread that evaluates it
    {
      T L[NV], F[NV];
      T *f = Fx + tj * LF + ti;
#pragma unroll
      for (int v = 0; v < NV; v++) L[v] = f[v * C::FACES];
      riemann<T, NDIM, 0, (SCH & kSchHLL) != 0>(L, xl, gamma, F);
#pragma unroll
      for (int v = 0; v < NV; v++) f[v * C::FACES] = F[v];
      if (I == 0) bflux(0, J, k, F);
      f = Fy + tj * LF + ti;
#pragma unroll
      for (int v = 0; v < NV; v++) L[v] = f[v * C::FACES];
      riemann<T, NDIM, 1, (SCH & kSchHLL) != 0>(L, yl, gamma, F);
#pragma unroll
      for (int v = 0; v < NV; v++) f[v * C::FACES] = F[v];
      if (J == 0) bflux(2, I, k, F);
    }
    if (extra && eup) {
      // y faces on exchanged velocities, so that both sides' lanes evaluate
      // an x-normal flux
      T *f = ey ? Fy + TS * LF + em : Fx + em * LF + TS;
      T L[NV], R[NV], F[NV];
#pragma unroll
      for (int v = 0; v < NV; v++) L[v] = f[v * C::FACES];
#pragma unroll
      for (int v = 0; v < NV; v++) R[v] = E[v];
      auto exchange = [&](T *a) {
        const T a1 = a[1], a2 = a[2];
        a[1] = ey ? a2 : a1;
        a[2] = ey ? a1 : a2;
      };
      exchange(L);
      exchange(R);
      riemann<T, NDIM, 0, (SCH & kSchHLL) != 0>(L, R, gamma, F);
      exchange(F);
#pragma unroll
      for (int v = 0; v < NV; v++) f[v * C::FACES] = F[v];
      if (!ey && i0 + TS == N) bflux(1, j0 + em, k, F);
      if (ey && j0 + TS == N) bflux(3, i0 + em, k, F);
    }
    __syncthreads();
    T Uout[NV];
    [[maybe_unused]] T src[NV];
    if constexpr ((SCH & kSchGravity) != 0) {
      T gm = T(0);
      src[0] = T(0);
#pragma unroll
      for (int d = 0; d < NDIM; d++) {
        src[1 + d] = U0[0] * (T)M.grav[d];
        gm += (T)M.grav[d] * U0[1 + d];
      }
      src[NV - 1] = gm;
    }
    [[maybe_unused]] T Up2[NV], Up3[NV];
    if constexpr (STG == 4) {
      loadc((const T *)M.s[role_buffer(ss.prev2, cur)] + b * bel + k * sk, Up2);
      loadc((const T *)M.s[role_buffer(ss.prev3, cur)] + b * bel + k * sk, Up3);
    }
    const auto ro = buf_rsrc(uo + k * sk);
#pragma unroll
    for (int v = 0; v < NV; v++) {
      const T *fx = Fx + v * C::FACES + tj * LF + ti, *fy = Fy + v * C::FACES + tj * LF + ti;
      T div = (fx[1] - fx[0]) + (fy[LF] - fy[0]);
      if constexpr (NDIM == 3) {
        div += Fz1[v] - Fz[v];
        Fz[v] = Fz1[v];
      }
      T base;
      if constexpr (STG == 1) base = U0[v];
      else if constexpr (STG == 2) base = T(0.5) * (Up[v] + U0[v]);
      else if constexpr (STG == 3) base = (T)ss.wp * Up[v] + (T)ss.wd * U0[v];
      else base = (((T)ss.wp * Up[v] + (T)ss.wp2 * Up2[v]) + (T)ss.wp3 * Up3[v]) + (T)ss.wd * U0[v];
      if constexpr ((SCH & kSchGravity) != 0) Uout[v] = (base + dts * src[v]) - cdt * div;
      else Uout[v] = base - cdt * div;
      buf_store<T>(Uout[v], ro, lo_b, (uint32_t)(v * sv * (int)sizeof(T)));
    }
    // cells next to F2C faces are finished (and their dt taken) by the flux fix
    if ((STG == 2 || (STG >= 3 && ss.epi)) && !(skip_xy || (skip_lo && k == 0) || (skip_hi && k == N - 1))) {
      if constexpr (sizeof(T) == 8) vloc = fmax(vloc, cell_inv_dt<NDIM>((const double *)Uout, M.gamma, dx, bad));
      else vloc = fmaxf(vloc, cell_inv_dt<NDIM>((const float *)Uout, (float)gamma, (float)idx, bad));
    }
    if constexpr (NDIM == 3) {
      if (k + 1 < k1) {
        T W[NV];
        to_prim<T, NDIM>(nx, gamma, W);
#pragma unroll
        for (int v = 0; v < NV; v++) {
#pragma unroll
          for (int s = 0; s < 4; s++) w[s][v] = w[s + 1][v];
          w[4][v] = W[v];
        }
      }
    }
  }
  if (STG == 2 || (STG >= 3 && ss.epi)) {
    vmax = fmax(vmax, (double)vloc);
    flush_dt(M, vmax, bad);
  }
}

template <typename T, int NDIM, int TS, int SCH>
static void launch_tiles(unsigned n, int kd, const MeshDev *d, int stage, const SubStep &ss, hipStream_t s) {
  switch (stage) {
    case 1: weno_kernel<T, NDIM, TS, SCH, 1><<<n, TS * TS, 0, s>>>(d, n, kd, ss); break;
    case 2: weno_kernel<T, NDIM, TS, SCH, 2><<<n, TS * TS, 0, s>>>(d, n, kd, ss); break;
    case 3: weno_kernel<T, NDIM, TS, SCH, 3><<<n, TS * TS, 0, s>>>(d, n, kd, ss); break;
    default: weno_kernel<T, NDIM, TS, SCH, 4><<<n, TS * TS, 0, s>>>(d, n, kd, ss); break;
  }
}

template <typename T, int NDIM, int SCH>
static void launch_sizes(int64_t nblocks, int N, int n_cu, const MeshDev *d, int stage, const SubStep &ss,
                         hipStream_t s) {
  const int ts = N == 8 ? 8 : 16;
  const int64_t tiles = nblocks * (N / ts) * (N / ts);
  const int kd = NDIM == 3 ? weno_planes(nblocks, N, n_cu) : N;
  const unsigned n = (unsigned)(tiles * (N / kd));
  if (ts == 8) launch_tiles<T, NDIM, 8, SCH>(n, kd, d, stage, ss, s);
  else launch_tiles<T, NDIM, 16, SCH>(n, kd, d, stage, ss, s);
}

// This file is compiled once per scheme (F4_SCHEME: HLL and gravity bits);
// the compile with F4_SCHEME = 0 also holds the dispatcher.
#ifndef F4_SCHEME
#define F4_SCHEME 0
#endif

template <int SCH>
hipError_t launch_weno_sch(const MeshDev *d, int64_t nblocks, int N, int n_cu, int stage, int ndim, bool f64,
                           hipStream_t s, const SubStep &ss) {
  if (f64) {
    if (ndim == 3) launch_sizes<double, 3, SCH>(nblocks, N, n_cu, d, stage, ss, s);
    else launch_sizes<double, 2, SCH>(nblocks, N, n_cu, d, stage, ss, s);
  } else {
    if (ndim == 3) launch_sizes<float, 3, SCH>(nblocks, N, n_cu, d, stage, ss, s);
    else launch_sizes<float, 2, SCH>(nblocks, N, n_cu, d, stage, ss, s);
  }
  return hipGetLastError();
}
template hipError_t launch_weno_sch<F4_SCHEME>(const MeshDev *, int64_t, int, int, int, int, bool, hipStream_t,
                                               const SubStep &);

#if F4_SCHEME == 0
#define F4_EXTERN_SCHEME(S) \
  extern template hipError_t launch_weno_sch<S>(const MeshDev *, int64_t, int, int, int, int, bool, hipStream_t, \
                                                const SubStep &);
F4_EXTERN_SCHEME(2)
F4_EXTERN_SCHEME(4)
F4_EXTERN_SCHEME(6)
#undef F4_EXTERN_SCHEME

hipError_t launch_weno_stage(const MeshDev *d_mesh, int64_t nblocks, int block_n, int n_cu, int stage, int ndim,
                             bool f64, int scheme, hipStream_t s, const SubStep &ss) {
  if (nblocks <= 0) return hipSuccess;
  switch (scheme & (kSchHLL | kSchGravity)) {
    case 0: return launch_weno_sch<0>(d_mesh, nblocks, block_n, n_cu, stage, ndim, f64, s, ss);
    case kSchHLL: return launch_weno_sch<kSchHLL>(d_mesh, nblocks, block_n, n_cu, stage, ndim, f64, s, ss);
    case kSchGravity: return launch_weno_sch<kSchGravity>(d_mesh, nblocks, block_n, n_cu, stage, ndim, f64, s, ss);
    default: return launch_weno_sch<kSchHLL | kSchGravity>(d_mesh, nblocks, block_n, n_cu, stage, ndim, f64, s, ss);
  }
}
#endif

}  // namespace f4
