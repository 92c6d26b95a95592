// Stage kernel of scalar advection (Sec. 3.4): one conserved variable rho
// carried by a uniform velocity v, rho_t + div(rho v) = 0.  The face values
// come from the mesh's reconstruction (minmod or van Leer MUSCL, WENO5), the
// physical flux on either side of a face is rho v_d, and the numerical flux
// (Rusanov or HLL with the wave speeds min(v_d, 0) and max(v_d, 0)) is upwind.
//
// One workgroup per block, or per slab of its planes where the blocks do not
// fill the chip, and one thread per (i, j) column, which marches along k.  Per
// plane the workgroup stages the plane with its x and y face halos in LDS (the interior from the threads' own z windows; the halo of a
// same-level face straight from the neighbouring block's interior when the
// mesh gathers halos, else - and always across refinement and boundary
// faces - from the block's stored ghosts, filled by the ghost rounds),
// double buffered so that one barrier per plane suffices; every thread then
// evaluates the two x faces and two y faces of its cell from LDS and the
// upper z face from its register window of the column (the lower one is the
// upper face of the previous plane).  The update, the refinement-face flux
// capture and the CFL epilogue follow the Euler stage kernels: stage 1 / 2
// Heun's stages, 3 the generic sub-step, 4 the generic sub-step with three
// earlier states.  A stage moves the state once in and once out, and Heun's
// second also reads U^n: two steps of 256^3 cells in FP32 move 671 MB, 143 us at
// the 4.7 TB/s of a large copy.  The kernel takes 205 us there (227 with two
// reconstructions per face), 70 % of that rate; the rest is its VALU work on the
// faces, the LDS rows and the addresses, and the halo lines.
// FP64 plain 335 us, WENO5 FP64 899 us (729 and 1985 with two reconstructions,
// whole blocks and halos from a ghost-fill pass).
#include <type_traits>

#include "device_common.h"
#include "foap4_internal.h"

namespace f4 {

// Reconstruction of an advection stage: LIM 0 minmod, 1 van Leer, 2 WENO5.
// R = cells on either side of a face that the stencil reaches.
template <int LIM>
struct AdvStencil {
  static constexpr int R = (LIM == 2) ? 3 : 2;
};

// Value at the right face of cell c2 of c0 .. c4 (WENO5 of Jiang and Shu,
// eps 1e-6, ideal weights 1/10, 6/10, 3/10).
template <typename T>
__device__ __forceinline__ T adv_weno5(T v0, T v1, T v2, T v3, T v4) {
  const T s6 = T(1) / T(6);
  const T q0 = (T(2) * v0 - T(7) * v1 + T(11) * v2) * s6;
  const T q1 = (-v1 + T(5) * v2 + T(2) * v3) * s6;
  const T q2 = (T(2) * v2 + T(5) * v3 - v4) * s6;
  const T c13 = T(13) / T(12), c14 = T(0.25);
  T a = v0 - T(2) * v1 + v2, b = v0 - T(4) * v1 + T(3) * v2;
  const T b0 = c13 * a * a + c14 * b * b;
  a = v1 - T(2) * v2 + v3;
  b = v1 - v3;
  const T b1 = c13 * a * a + c14 * b * b;
  a = v2 - T(2) * v3 + v4;
  b = T(3) * v2 - T(4) * v3 + v4;
  const T b2 = c13 * a * a + c14 * b * b;
  const T e0 = T(1e-6) + b0, e1 = T(1e-6) + b1, e2 = T(1e-6) + b2;
  const T a0 = fdiv(T(0.1), e0 * e0), a1 = fdiv(T(0.6), e1 * e1), a2 = fdiv(T(0.3), e2 * e2);
  return fdiv(a0 * q0 + a1 * q1 + a2 * q2, a0 + a1 + a2);
}

// Value of cell `at` (relative) at its face in direction DIR (+1: upper), get(k)
// the cell k cells above.
template <typename T, int LIM, int DIR, typename Get>
__device__ __forceinline__ T adv_value(Get get, int at) {
  const T b = get(at - DIR), c = get(at), d = get(at + DIR);
  if constexpr (LIM == 2) return adv_weno5(T(get(at - 2 * DIR)), b, c, d, T(get(at + 2 * DIR)));
  else return c + T(0.5) * limit<LIM>(c - b, d - c);
}

// Numerical flux through the upper face of cell 0, velocity component v (the
// same on the whole mesh), get(k) the cell k cells above.  Rusanov's flux
// (v L + v R)/2 - |v| (R - L)/2 (the largest of |min(v, 0)| and |max(v, 0)| is
// |v|) and HLL with s0 = min(v, 0), s1 = max(v, 0) are both the upwind flux,
// v L for v >= 0 and v R below: one reconstruction per face, not two.  (A NaN
// or infinite cell then reaches only its downwind neighbours.)
template <typename T, int LIM, typename Get>
__device__ __forceinline__ T adv_flux(Get get, T v) {
  return v * (v >= T(0) ? adv_value<T, LIM, 1>(get, 0) : adv_value<T, LIM, -1>(get, 1));
}

// Stores the refinement-face flux F of face f at in-face position (t1, t2)
// (layout [slot][t2][t1], one variable).
template <typename T, int NDIM>
__device__ __forceinline__ void adv_bflux(const MeshDev &M, int info, int t1, int t2, T F) {
  if (info < 0) return;
  const int N = M.N;
  T *buf = (T *)((info & 1) ? M.bflux_c : M.bflux_f);
  const int64_t slot = info >> 1;
  const int64_t o = (NDIM == 3) ? (slot * N + t2) * N + t1 : slot * N + t1;
  gstore(buf + o, F);
}

// LDS elements: two planes of (N + 2g)^2 cells.
__host__ __device__ constexpr int adv_lds(int N, int g) { return 2 * (N + 2 * g) * (N + 2 * g); }

// MAXT: the largest workgroup (N^2 threads) the instantiation serves: 1024
// for 32^2 columns, 256 for 8^2 and 16^2 (which leaves the compiler up to 512
// registers per thread instead of 128).  HS: halo cells per thread and
// plane, ceil(4 g N / N^2): 1, or 2 for 8^2 columns with g >= 3 (N >= 2 g
// bounds it by 2).  Eight waves per SIMD asked of the compiler for FP32 MUSCL
// gained 10 % on 8^3 blocks and lost 4 % on 256^3 cells (205 -> 213 us).
template <typename T, int NDIM, int LIM, int STG, int MAXT, int HS, bool SLABS>
__global__ __launch_bounds__(MAXT) void advect_kernel(const MeshDev *__restrict__ Mp, int lslabs, SubStep ss) {
  constexpr int R = AdvStencil<LIM>::R;
  extern __shared__ __align__(16) unsigned char adv_smem[];
  const MeshDev &M = *Mp;
  const int N = M.N, g = M.g, P = N + 2 * g, Q = P;
  const int rows = (NDIM == 3) ? P * P : P;  // rows (k, j) of the row part of a block
  const int64_t sv = (NDIM == 3) ? (int64_t)P * P * P : (int64_t)P * P;
  // XCD-aware order: workgroup w runs on XCD w mod 8, so XCD x is given the
  // contiguous range of (block, slab) items [x q + min(x, r), ...) of q or q + 1
  // items (8 q + r in all): blocks that are neighbours in Morton order, whose
  // face halos each reads, share that XCD's L2.  A bijection onto all items.
  const int64_t all = SLABS ? M.nb << lslabs : M.nb, xq = all / 8, xr = all % 8;
  const int64_t xid = blockIdx.x % 8, xi = blockIdx.x / 8;
  const int64_t item = xid * xq + (xid < xr ? xid : xr) + xi;
  // slabs of N >> lslabs planes per block
  const int64_t b = SLABS ? item >> lslabs : item;
  const int kd = SLABS ? N >> lslabs : (NDIM == 3) ? N : 1;
  const int k0 = SLABS ? (int)(item & ((1 << lslabs) - 1)) * kd : 0, k1 = k0 + kd;
  const int t = threadIdx.x, i = t % N, j = t / N;
  const int cur = M.cur;
  const int64_t boff = b * sv;
  const T *ud0 = (const T *)M.s[STG >= 3 ? role_buffer(ss.deriv, cur) : (STG == 1 ? cur : 1 - cur)];
  const T *ud = ud0 + boff;
  T *uo = (T *)M.s[STG >= 3 ? role_buffer(ss.out, cur) : (STG == 1 ? 1 - cur : cur)] + boff;
  const T *up = (const T *)M.s[STG >= 3 ? role_buffer(ss.prev, cur) : cur] + boff;
  const double dx = ldexp(M.dx0, -gload(M.level + b));
  const T idx = (T)(1.0 / dx);
  const double dt = gload(M.scal + kDt);
  const T dts = (T)(STG >= 3 ? ss.c * dt : (STG == 1 ? dt : 0.5 * dt));
  const T cdt = dts * idx;
  int finfo[2 * NDIM];
  // with gathered halos, the block data of the same-level neighbour across
  // each face (null: the face's halo comes from this block's stored ghosts)
  const T *nbp[2 * NDIM];
#pragma unroll
  for (int f = 0; f < 2 * NDIM; f++) {
    finfo[f] = gload(M.face_info + b * 2 * NDIM + f);
    nbp[f] = (M.gather && finfo[f] <= -2) ? ud0 + (int64_t)(-2 - finfo[f]) * sv : nullptr;
  }
  const T vx = (T)M.vel[0], vy = (T)M.vel[1], vz = (T)M.vel[2];
  T *lds = (T *)adv_smem;
  // halo cells of one plane: the 2g y-ghost rows (x inside) and the 2g
  // x-ghosts of the N interior rows
  const int nhalo = 4 * g * N;
  auto row_of = [&](int jj, int kk) { return (NDIM == 3) ? (kk + g) * P + (jj + g) : (jj + g); };
  // a cell of the block or of its face halo (at most one coordinate outside
  // 0 .. N-1): across a same-level face from the neighbour's interior when
  // gathering, else from the stored ghosts
  auto cell = [&](int x, int y, int kk) -> T {
    if (x < 0) return nbp[0] ? gload(nbp[0] + row_of(y, kk) * N + x + N) : gload(ud + rows * N + row_of(y, kk) * 2 * g + x + g);
    if (x >= N) return nbp[1] ? gload(nbp[1] + row_of(y, kk) * N + x - N) : gload(ud + rows * N + row_of(y, kk) * 2 * g + x - N + g);
    const T *src = ud;
    if (y < 0 && nbp[2]) { src = nbp[2]; y += N; }
    else if (y >= N && nbp[3]) { src = nbp[3]; y -= N; }
    if constexpr (NDIM == 3) {
      if (kk < 0 && nbp[4]) { src = nbp[4]; kk += N; }
      else if (kk >= N && nbp[5]) { src = nbp[5]; kk -= N; }
    }
    return gload(src + row_of(y, kk) * N + x);
  };
  // this thread's halo cells of a plane (the same (x, y) in every plane)
  constexpr int HMAX = HS;
  int hx[HMAX], hy[HMAX];
  bool hv[HMAX];
#pragma unroll
  for (int q = 0; q < HMAX; q++) {
    const int h = t + q * N * N;
    hv[q] = h < nhalo;
    if (h < 2 * g * N) {  // y ghost rows: y = -g .. -1, N .. N + g - 1
      const int r = h / N;
      hx[q] = h % N;
      hy[q] = r < g ? r - g : N + r - g;
    } else {              // x ghosts of rows 0 .. N-1, c = 0 .. 2g-1
      const int e = h - 2 * g * N, cc = e % (2 * g);
      hy[q] = e / (2 * g);
      hx[q] = cc < g ? cc - g : N + cc - g;
    }
  }
  // Loads run D planes ahead of use: with one variable a plane holds little
  // work, so the window cells, halo cells and earlier-state cells of the next
  // D planes are in flight together (in register slots: plane kk in slot
  // kk % D; the plane loop is unrolled by D so that every slot is named by a
  // constant).  FP64 workgroups of 1024 threads (128 registers) keep D = 2,
  // or D = 1 with WENO5.
  constexpr int D = (sizeof(T) == 8 && MAXT > 256) ? (LIM == 2 ? 1 : 2) : 4;
  const T *up2 = (const T *)M.s[STG == 4 ? role_buffer(ss.prev2, cur) : cur] + boff;
  const T *up3 = (const T *)M.s[STG == 4 ? role_buffer(ss.prev3, cur) : cur] + boff;
  // Addresses: cell (i, j, kk) of the own column is at the wave-uniform
  // plane base wbase(kk) (this block, or across -z / +z the neighbour's when
  // gathering) plus the lane's byte offset lo, read and written through
  // buffer descriptors; a halo cell of this thread is at hp[q] + kk hs[q].
  const int pstride = (NDIM == 3) ? P * N : 0;  // elements per plane of the row part
  const uint32_t lo = (uint32_t)(row_of(j, 0) * N + i) * (uint32_t)sizeof(T);
  auto wbase = [&](int kk) -> const T * {
    if constexpr (NDIM == 3) {
      if (kk < 0 && nbp[4]) return nbp[4] + (kk + N) * pstride;
      if (kk >= N && nbp[5]) return nbp[5] + (kk - N) * pstride;
    }
    return ud + kk * pstride;
  };
  const T *hp[HMAX];
  int hs[HMAX];
#pragma unroll
  for (int q = 0; q < HMAX; q++) {
    const int x = hx[q], y = hy[q];
    hp[q] = ud;
    hs[q] = 0;
    if (!hv[q]) continue;
    if (x < 0 || x >= N) {
      const T *nb = nbp[x < 0 ? 0 : 1];
      if (nb) {
        hp[q] = nb + row_of(y, 0) * N + (x < 0 ? x + N : x - N);
        hs[q] = pstride;
      } else {  // stored x ghosts: rows of 2 g after the row part
        hp[q] = ud + rows * N + row_of(y, 0) * 2 * g + (x < 0 ? x + g : x - N + g);
        hs[q] = (NDIM == 3) ? P * 2 * g : 0;
      }
    } else {
      const T *src = ud;
      int yy = y;
      if (y < 0 && nbp[2]) { src = nbp[2]; yy += N; }
      else if (y >= N && nbp[3]) { src = nbp[3]; yy -= N; }
      hp[q] = src + row_of(yy, 0) * N + x;
      hs[q] = pstride;
    }
  }
  T hq[D][HMAX], pq[D], pq2[D], pq3[D], wq[D];
  auto fetch = [&](int kk, auto slot) {  // the values plane kk needs beyond the window
    constexpr int S = decltype(slot)::value;
#pragma unroll
    for (int q = 0; q < HMAX; q++)
      if (hv[q]) hq[S][q] = gload(hp[q] + kk * hs[q]);
    if constexpr (STG >= 2) pq[S] = buf_load<T>(buf_rsrc(up + kk * pstride), lo, 0);
    if constexpr (STG == 4) {
      pq2[S] = buf_load<T>(buf_rsrc(up2 + kk * pstride), lo, 0);
      pq3[S] = buf_load<T>(buf_rsrc(up3 + kk * pstride), lo, 0);
    }
    wq[S] = buf_load<T>(buf_rsrc(wbase((NDIM == 3) ? kk + R : 0)), lo, 0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  // the z window of column (i, j): cells k - R + 1 .. k + R (3-D)
  T w[2 * R];
  if constexpr (NDIM == 3) {
#pragma unroll
    for (int s = 1; s < 2 * R; s++) w[s] = cell(i, j, k0 + s - R);
  }
  fetch(k0, I0{});
  if constexpr (D > 1) {
    if (k0 + 1 < k1) fetch(k0 + 1, I1{});
  }
  if constexpr (D > 2) {
    if (k0 + 2 < k1) fetch(k0 + 2, I2{});
    if (k0 + 3 < k1) fetch(k0 + 3, I3{});
  }
  T Fz = T(0);  // flux through the lower z face of the current plane
  // fluxes through a cell's lower and upper face (one test of the sign)
  auto pair = [&](auto get, T v, T &fm, T &fp) __attribute__((always_inline)) {
    if (v >= T(0)) {
      fm = v * adv_value<T, LIM, 1>(get, -1);
      fp = v * adv_value<T, LIM, 1>(get, 0);
    } else {
      fm = v * adv_value<T, LIM, -1>(get, 0);
      fp = v * adv_value<T, LIM, -1>(get, 1);
    }
  };
  auto plane = [&](const int k, auto slot) __attribute__((always_inline)) {
    constexpr int S = decltype(slot)::value;
    T *pl = lds + (k & 1) * Q * Q;  // cell (x, y) at (y + g) Q + x + g
    T c;
    if constexpr (NDIM == 3) {
#pragma unroll
      for (int s = 0; s < 2 * R - 1; s++) w[s] = w[s + 1];
      w[2 * R - 1] = wq[S];
      c = w[R - 1];
    } else {
      c = wq[S];
    }
    pl[(j + g) * Q + i + g] = c;
#pragma unroll
    for (int q = 0; q < HMAX; q++)
      if (hv[q]) pl[(hy[q] + g) * Q + hx[q] + g] = hq[S][q];
    const T cp = (STG >= 2) ? pq[S] : T(0);
    const T cp2 = (STG == 4) ? pq2[S] : T(0), cp3 = (STG == 4) ? pq3[S] : T(0);
    if (k + D < k1) fetch(k + D, slot);
    __syncthreads();
    // x faces i - 1/2 and i + 1/2, then y faces, from the staged plane
    const T *own = pl + (j + g) * Q + i + g;
    T fxm, fxp, fym, fyp;
    pair([&](int s) { return s == 0 ? c : own[s]; }, vx, fxm, fxp);
    T div = fxp - fxm;
    if (i == 0) adv_bflux<T, NDIM>(M, finfo[0], j, k, fxm);
    if (i == N - 1) adv_bflux<T, NDIM>(M, finfo[1], j, k, fxp);
    pair([&](int s) { return s == 0 ? c : own[s * Q]; }, vy, fym, fyp);
    div += fyp - fym;
    if (j == 0) adv_bflux<T, NDIM>(M, finfo[2], i, k, fym);
    if (j == N - 1) adv_bflux<T, NDIM>(M, finfo[3], i, k, fyp);
    if constexpr (NDIM == 3) {
      if (k == k0) {  // the slab's lower z face, from cells k0 - R .. k0 + R - 1
        T w0[2 * R];
        w0[0] = cell(i, j, k0 - R);
#pragma unroll
        for (int s = 1; s < 2 * R; s++) w0[s] = w[s - 1];
        Fz = adv_flux<T, LIM>([&](int s) { return w0[s + R - 1]; }, vz);
        if (k0 == 0) adv_bflux<T, NDIM>(M, finfo[4], i, j, Fz);
      }
      const T fzp = adv_flux<T, LIM>([&](int s) { return w[s + R - 1]; }, vz);
      div += fzp - Fz;
      if (k == N - 1) adv_bflux<T, NDIM>(M, finfo[5], i, j, fzp);
      Fz = fzp;
    }
    T base;
    if constexpr (STG == 1) base = c;
    else if constexpr (STG == 2) base = T(0.5) * (cp + c);
    else if constexpr (STG == 3) base = (T)ss.wp * cp + (T)ss.wd * c;
    else base = (((T)ss.wp * cp + (T)ss.wp2 * cp2) + (T)ss.wp3 * cp3) + (T)ss.wd * c;
    const T out = base - cdt * div;
    buf_store<T>(out, buf_rsrc(uo + k * pstride), lo, 0);
    if (STG == 2 || (STG >= 3 && ss.epi)) {
      // the CFL limit of advection is the same in every cell of the block;
      // only the state's finiteness is per cell (cells next to F2C faces
      // are checked after the flux fix)
      if (!isfinite(out)) atomic_max_pos(&M.scal[kBad], 1.0);
    }
  };
  for (int k = k0; k < k1; k += D) {
    plane(k, I0{});
    if constexpr (D > 1) {
      if (k + 1 >= k1) break;
      plane(k + 1, I1{});
    }
    if constexpr (D > 2) {
      if (k + 2 >= k1) break;
      plane(k + 2, I2{});
      if (k + 3 >= k1) break;
      plane(k + 3, I3{});
    }
  }
  if ((STG == 2 || (STG >= 3 && ss.epi)) && t == 0) {
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < NDIM; d++) s += fabs(M.vel[d]) / dx;
    atomic_max_pos_if_larger(&M.scal[kMaxInv], s);
  }
}

template <typename T, int NDIM, int LIM>
static void launch_adv(int64_t nb, int N, int g, int n_cu, const MeshDev *d, int stage, const SubStep &ss,
                       hipStream_t s) {
  const unsigned threads = (unsigned)(N * N);
  // slabs are a variant of their own, because their bounds cost registers that
  // whole blocks need (256^3 cells: 197 and 214 us)
  const int ls = NDIM == 3 ? advect_log2_slabs(nb, N, n_cu) : 0;
  const unsigned grid = (unsigned)(nb << ls);
  const size_t lds = (size_t)adv_lds(N, g) * sizeof(T);
#define F4_ADV(STG, MAXT, HS)                                                                                 \
  do {                                                                                                       \
    if (NDIM == 3 && ls > 0)                                                                                 \
      advect_kernel<T, NDIM, LIM, STG, MAXT, HS, NDIM == 3><<<grid, threads, lds, s>>>(d, ls, ss);           \
    else                                                                                                     \
      advect_kernel<T, NDIM, LIM, STG, MAXT, HS, false><<<grid, threads, lds, s>>>(d, 0, ss);                \
  } while (0)
#define F4_ADV_STAGES(MAXT, HS)                \
  switch (stage) {                             \
    case 1: F4_ADV(1, MAXT, HS); break;        \
    case 2: F4_ADV(2, MAXT, HS); break;        \
    case 3: F4_ADV(3, MAXT, HS); break;        \
    default: F4_ADV(4, MAXT, HS); break;       \
  }
  // halo cells of a plane: 4 g N (2-D: also 4 g N per row of planes)
  const bool two_halo = 4 * g * N > N * N;
  if (threads > 256) {
    F4_ADV_STAGES(1024, 1)  // N = 32 with g <= 4: 4 g N <= N^2
  } else if (two_halo) {
    F4_ADV_STAGES(256, 2)
  } else {
    F4_ADV_STAGES(256, 1)
  }
#undef F4_ADV_STAGES
#undef F4_ADV
}

template <typename T, int NDIM>
static void launch_adv_limiter(int64_t nb, int N, int g, int n_cu, const MeshDev *d, int stage, int limiter,
                               const SubStep &ss, hipStream_t s) {
  if (limiter == FOAP4_LIM_WENO5) launch_adv<T, NDIM, 2>(nb, N, g, n_cu, d, stage, ss, s);
  else if (limiter == FOAP4_LIM_VANLEER) launch_adv<T, NDIM, 1>(nb, N, g, n_cu, d, stage, ss, s);
  else launch_adv<T, NDIM, 0>(nb, N, g, n_cu, d, stage, ss, s);
}

hipError_t launch_advect_stage(const MeshDev *d_mesh, int64_t nblocks, int block_n, int n_ghost, int n_cu, int stage,
                               int ndim, bool f64, int limiter, hipStream_t s, const SubStep &ss) {
  if (nblocks <= 0) return hipSuccess;
  const int64_t nb = nblocks;
  if (f64) {
    if (ndim == 3) launch_adv_limiter<double, 3>(nb, block_n, n_ghost, n_cu, d_mesh, stage, limiter, ss, s);
    else launch_adv_limiter<double, 2>(nb, block_n, n_ghost, n_cu, d_mesh, stage, limiter, ss, s);
  } else {
    if (ndim == 3) launch_adv_limiter<float, 3>(nb, block_n, n_ghost, n_cu, d_mesh, stage, limiter, ss, s);
    else launch_adv_limiter<float, 2>(nb, block_n, n_ghost, n_cu, d_mesh, stage, limiter, ss, s);
  }
  return hipGetLastError();
}

}  // namespace f4
