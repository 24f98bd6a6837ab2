// HIP kernels of the OEFE operator application Ht X = M^-1/2 H M^-1/2 X and the
// scaled Chebyshev recurrence step built on it (gfx950, wave64).
//
// One operator step (out = alpha (Ht x - c x) - beta prev) is:
//   1. zo       Z^O = S X^O                                   (small dense)
//   2. cell     per cell: z_e = m^-1/2 (theta o X)|_e, y_e = K_e z_e + B^T diag(W V) B z_e
//               (sum-factorized, see fe_cell_kernel) -> node-slot grid
//   3. node     per FE node: fixed-order sum of the (up to 8) cell results sharing it
//               (no atomics), times m^-1/2, + (m^-1/2 H^co) Z^O, recurrence epilogue; per 64-row
//               tile the partial conj(m^-1/2 H^co)^T X over its rows (in a recurrence, of the X
//               that this step writes)
//   4. reduce   W' = sum of the tile partials of each function (fixed order)
//   5. gemm     W' += H^oo Z^O ;  enrichment rows alpha (S W' - c x) - beta prev
// Every launch can cover several operators of one mesh at once (k-points): the
// per-operator arguments travel in a KBatch and blockIdx.z selects the operator.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "oefe_kernels.h"

namespace oefe {

namespace {

template <typename T>
struct C2 {
  T r, i;
};
template <typename T>
__device__ __forceinline__ C2<T> cmul(C2<T> a, C2<T> b) {
  return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r};
}
template <typename T>
__device__ __forceinline__ C2<T> cjmul(C2<T> a, C2<T> b) {  // conj(a) * b
  return {a.r * b.r + a.i * b.i, a.r * b.i - a.i * b.r};
}

template <typename T>
struct Phase3 {
  T re[3], im[3];
};

constexpr int KMAX = 8;  // operators per batched launch

// Per-operator arguments of one recurrence step (leading dimensions in elements of T).
template <typename T>
struct KP {
  const T* x;
  const T* prev;
  T* out;
  int64_t ldx, ldo;
  int nv, ncr;  // vectors (complex elements when complex) and real columns
  T* ycell;
  int ldc;
  T* zo;  // Z^O of this step
  T* zn;  // Z^O of the next one (a recurrence)
  T* part;
  T* part2;
  int nch;  // chunks per function in part2
  T* wp;
  double* pq;  // one real column: receives x . out (null: not wanted), and its partials per node workgroup
  double* pq_part;
  const T* wv;  // W (V + the form's constant shift) of this operator at its quadrature points
  const T* tv;
  const T* S;
  const T* Hoo;
  T alpha, c, beta;
  const double* sc;  // device (alpha, c, beta) of the step in place of the three above, or null
  Phase3<T> ph;
  T uk[3];  // periodic-function k-point form: (h/2)^3 (2/h) k_d (zero otherwise)
};

// the step's scalars: from device memory when the filter's bounds live on the device
template <typename T>
__device__ __forceinline__ void step_scalars(const KP<T>& P, T& alpha, T& c, T& beta) {
  if (P.sc) {
    alpha = (T)P.sc[0];
    c = (T)P.sc[1];
    beta = (T)P.sc[2];
  } else {
    alpha = P.alpha;
    c = P.c;
    beta = P.beta;
  }
}

template <typename T>
struct KBatch {
  int nk;
  KP<T> k[KMAX];
};


// ---------------------------------------------------------------------------
// 1D passes of the sum-factorized cell operator, shared by the cell kernels so that every
// launch shape does the same arithmetic.  EO (degree 4): each 5-point contraction through
// the even and odd halves of its matrix (EO5); otherwise plain sums in index order.
// ---------------------------------------------------------------------------
// out(q, (M v)_q) for q < 5 from in(a) = v_a, M given by its halves
template <typename T, typename In, typename Out>
__device__ __forceinline__ void eo5_apply(const EO5<T>& m, In in, Out out) {
  const T v0 = in(0), v1 = in(1), v2 = in(2), v3 = in(3), v4 = in(4);
  const T e0 = v0 + v4, e1 = v1 + v3, o0 = v0 - v4, o1 = v1 - v3;
  const T E0 = m.e[0][0] * e0 + m.e[0][1] * e1 + m.e[0][2] * v2;
  const T E1 = m.e[1][0] * e0 + m.e[1][1] * e1 + m.e[1][2] * v2;
  const T E2 = m.e[2][0] * e0 + m.e[2][1] * e1 + m.e[2][2] * v2;
  const T O0 = m.o[0][0] * o0 + m.o[0][1] * o1;
  const T O1 = m.o[1][0] * o0 + m.o[1][1] * o1;
  out(0, E0 + O0);
  out(1, E1 + O1);
  out(2, E2);
  out(3, E1 - O1);
  out(4, E0 - O0);
}

// x- then y-pass with B1 on a z-plane: v[ay][ax] -> v[qy][qx] (t is scratch)
template <typename T, int P1, bool EO>
__device__ __forceinline__ void cell_pass_xy(const CellCoef<T>& cf, T (&v)[P1 * P1], T (&t)[P1 * P1]) {
  if constexpr (EO) {
#pragma unroll
    for (int ay = 0; ay < P1; ++ay)
      eo5_apply(cf.eB1, [&](int a) { return v[ay * P1 + a]; }, [&](int q, T r) { t[ay * P1 + q] = r; });
#pragma unroll
    for (int qx = 0; qx < P1; ++qx)
      eo5_apply(cf.eB1, [&](int a) { return t[a * P1 + qx]; }, [&](int q, T r) { v[q * P1 + qx] = r; });
  } else {
#pragma unroll
    for (int ay = 0; ay < P1; ++ay)
#pragma unroll
      for (int qx = 0; qx < P1; ++qx) {
        T s = 0;
#pragma unroll
        for (int ax = 0; ax < P1; ++ax) s += cf.B1[qx][ax] * v[ay * P1 + ax];
        t[ay * P1 + qx] = s;
      }
#pragma unroll
    for (int qy = 0; qy < P1; ++qy)
#pragma unroll
      for (int qx = 0; qx < P1; ++qx) {
        T s = 0;
#pragma unroll
        for (int ay = 0; ay < P1; ++ay) s += cf.B1[qy][ay] * t[ay * P1 + qx];
        v[qy * P1 + qx] = s;
      }
  }
}

// z-pass with B1 on an x-plane: t[az][qy] -> u[qz][qy]
template <typename T, int P1, bool EO>
__device__ __forceinline__ void cell_pass_z(const CellCoef<T>& cf, const T (&t)[P1 * P1], T (&u)[P1 * P1]) {
  if constexpr (EO) {
#pragma unroll
    for (int qy = 0; qy < P1; ++qy)
      eo5_apply(cf.eB1, [&](int a) { return t[a * P1 + qy]; }, [&](int q, T r) { u[q * P1 + qy] = r; });
  } else {
#pragma unroll
    for (int qz = 0; qz < P1; ++qz)
#pragma unroll
      for (int qy = 0; qy < P1; ++qy) {
        T s = 0;
#pragma unroll
        for (int az = 0; az < P1; ++az) s += cf.B1[qz][az] * t[az * P1 + qy];
        u[qz * P1 + qy] = s;
      }
  }
}

// t' = (B^T)_y (B^T)_z t: t[qz][qy] -> tp[az][ay] (v is scratch)
template <typename T, int P1, bool EO>
__device__ __forceinline__ void cell_back_yz(const CellCoef<T>& cf, const T (&t)[P1 * P1], T (&v)[P1 * P1],
                                             T (&tp)[P1 * P1]) {
  if constexpr (EO) {
#pragma unroll
    for (int qz = 0; qz < P1; ++qz)
      eo5_apply(cf.eB1t, [&](int q) { return t[qz * P1 + q]; }, [&](int ay, T r) { v[qz * P1 + ay] = r; });
#pragma unroll
    for (int ay = 0; ay < P1; ++ay)
      eo5_apply(cf.eB1t, [&](int q) { return v[q * P1 + ay]; }, [&](int az, T r) { tp[az * P1 + ay] = r; });
  } else {
#pragma unroll
    for (int qz = 0; qz < P1; ++qz)
#pragma unroll
      for (int ay = 0; ay < P1; ++ay) {
        T s = 0;
#pragma unroll
        for (int qy = 0; qy < P1; ++qy) s += cf.B1[qy][ay] * t[qz * P1 + qy];
        v[qz * P1 + ay] = s;
      }
#pragma unroll
    for (int az = 0; az < P1; ++az)
#pragma unroll
      for (int ay = 0; ay < P1; ++ay) {
        T s = 0;
#pragma unroll
        for (int qz = 0; qz < P1; ++qz) s += cf.B1[qz][az] * v[qz * P1 + ay];
        tp[az * P1 + ay] = s;
      }
  }
}

// the x kinetic term before its x-pass: u <- kappa (B^T W)_y (B^T W)_z u (v is scratch)
template <typename T, int P1, bool EO>
__device__ __forceinline__ void cell_xkin_yz(const CellCoef<T>& cf, T (&u)[P1 * P1], T (&v)[P1 * P1]) {
  if constexpr (EO) {
#pragma unroll
    for (int qz = 0; qz < P1; ++qz)
      eo5_apply(cf.eBtW, [&](int q) { return u[qz * P1 + q]; }, [&](int ay, T r) { v[qz * P1 + ay] = r; });
#pragma unroll
    for (int ay = 0; ay < P1; ++ay)
      eo5_apply(cf.ekBtW, [&](int q) { return v[q * P1 + ay]; }, [&](int az, T r) { u[az * P1 + ay] = r; });
  } else {
#pragma unroll
    for (int qz = 0; qz < P1; ++qz)
#pragma unroll
      for (int ay = 0; ay < P1; ++ay) {
        T s = 0;
#pragma unroll
        for (int qy = 0; qy < P1; ++qy) s += cf.BtW[ay][qy] * u[qz * P1 + qy];
        v[qz * P1 + ay] = s;
      }
#pragma unroll
    for (int az = 0; az < P1; ++az)
#pragma unroll
      for (int ay = 0; ay < P1; ++ay) {
        T s = 0;
#pragma unroll
        for (int qz = 0; qz < P1; ++qz) s += cf.BtW[az][qz] * v[qz * P1 + ay];
        u[az * P1 + ay] = cf.kappa * s;
      }
  }
}

// the quadrature-point terms: t = W V u + kappa w_x (w_z L1_y u + w_y L1_z u); wvq(qz, qy) is
// W V at the point (qx, qy, qz) of this plane
template <typename T, int P1, bool EO, typename WV>
__device__ __forceinline__ void cell_point_terms(const CellCoef<T>& cf, const T (&u)[P1 * P1], T (&t)[P1 * P1],
                                                 WV wvq, T kx) {
#pragma unroll
  for (int qz = 0; qz < P1; ++qz) {
    T ly[P1];
    if constexpr (EO) {
      eo5_apply(cf.eL1, [&](int k) { return u[qz * P1 + k]; }, [&](int q, T r) { ly[q] = r; });
    } else {
#pragma unroll
      for (int qy = 0; qy < P1; ++qy) {
        T s = 0;
#pragma unroll
        for (int k = 0; k < P1; ++k) s += cf.L1[qy][k] * u[qz * P1 + k];
        ly[qy] = s;
      }
    }
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) {
      T lz = 0;
#pragma unroll
      for (int k = 0; k < P1; ++k) lz += cf.L1[qz][k] * u[k * P1 + qy];
      t[qz * P1 + qy] = wvq(qz, qy) * u[qz * P1 + qy] + kx * (cf.w[qz] * ly[qy] + cf.w[qy] * lz);
    }
  }
}

// x-pass with B^T of one row: y[ax] = sum_q B1[q][ax] r[q]
template <typename T, int P1, bool EO>
__device__ __forceinline__ void cell_back_x(const CellCoef<T>& cf, const T (&r)[P1], T* y) {
  if constexpr (EO) {
    eo5_apply(cf.eB1t, [&](int q) { return r[q]; }, [&](int ax, T o) { y[ax] = o; });
  } else {
#pragma unroll
    for (int ax = 0; ax < P1; ++ax) {
      T s = 0;
#pragma unroll
      for (int q = 0; q < P1; ++q) s += cf.B1[q][ax] * r[q];
      y[ax] = s;
    }
  }
}

// ---------------------------------------------------------------------------
// Cell kernel.
//
// Workgroup = P1 waves; wave w owns "plane" w of the (p+1)^3 cell tensor, lane l
// owns column l of a 64-column tile (CPT = 64 / CW cells x CW real columns).
// The x- and y-direction 1D passes run in registers on z-planes; a transpose
// through LDS gives x-planes for the z-pass and the quadrature-point work.
// In quadrature space the cell operator is
//   t = W V u + kappa [ (W (x) L1 (x) W) + (W (x) W (x) L1) ] u      (y-, z- kinetic terms)
//   y = B^T t + kappa (B^T L1) (x) (B^T W) (x) (B^T W) u                (x kinetic term)
// with u = B z, L1 the Gauss-point collocation Laplacian, kappa = h/4, which
// equals K_e z + B^T diag(W V) B z with the exact (Gauss) cell stiffness.
// ---------------------------------------------------------------------------
template <typename T, int P1, int CW, bool CPLX>
__global__ __launch_bounds__(64 * P1) void fe_cell_kernel(KBatch<T> kb, CellCoef<T> cf, int nc, int p, int n,
                                                          int64_t n_cells) {
  constexpr int NP = P1 * P1;
  constexpr int CPT = 64 / CW;
  constexpr bool EO = P1 == 5;  // the same passes as the planes-in-lanes kernel
  __shared__ T lds[NP * P1][64];
  const KP<T>& P = kb.k[blockIdx.z];
  const int ncr = P.ncr;
  if ((int)blockIdx.y * CW >= ncr) return;  // column block beyond this operator's width
  const T* __restrict__ X = P.x;
  const int64_t ldx = P.ldx;
  T* __restrict__ Yc = P.ycell;
  const int ldc = P.ldc;
  const Phase3<T> ph = P.ph;
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int cl = lane / CW, col = lane % CW;
  const int64_t e = (int64_t)blockIdx.x * CPT + cl;
  const int j = blockIdx.y * CW + col;
  const bool valid = (e < n_cells) && (j < ncr);
  const int64_t ee = valid ? e : 0;
  const int cx = (int)(ee % nc), cy = (int)((ee / nc) % nc), cz = (int)(ee / ((int64_t)nc * nc));

  // 1. gather plane az = w with the m^-1/2 pre-scale (and Bloch phase)
  T v[NP];
  {
    const int az = w;
    int iz = cz * p + az;
    bool wz = iz >= n;
    if (wz) iz -= n;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int iy = cy * p + ay;
      bool wy = iy >= n;
      if (wy) iy -= n;
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int ix = cx * p + ax;
        bool wx = ix >= n;
        if (wx) ix -= n;
        const int64_t g = ix + (int64_t)n * (iy + (int64_t)n * iz);
        const T sc = cf.mscale * cf.om[ax] * cf.om[ay] * cf.om[az];
        T val = 0;
        if (valid) {
          if constexpr (!CPLX) {
            val = X[g * ldx + j];
          } else {
            const T* px = X + g * ldx + (j & ~1);
            C2<T> z{px[0], px[1]};
            if (wx) z = cmul(z, C2<T>{ph.re[0], ph.im[0]});
            if (wy) z = cmul(z, C2<T>{ph.re[1], ph.im[1]});
            if (wz) z = cmul(z, C2<T>{ph.re[2], ph.im[2]});
            val = (j & 1) ? z.i : z.r;
          }
        }
        v[ay * P1 + ax] = sc * val;
      }
    }
  }
  // 2. x- then y-pass with B1 (in registers)
  T t[NP];
  cell_pass_xy<T, P1, EO>(cf, v, t);
  // 3. transpose z-planes -> x-planes: lds[(az*P1 + qy)*P1 + qx]
#pragma unroll
  for (int qy = 0; qy < P1; ++qy)
#pragma unroll
    for (int qx = 0; qx < P1; ++qx) lds[(w * P1 + qy) * P1 + qx][lane] = v[qy * P1 + qx];
  __syncthreads();
  // this wave now owns qx = w; u[az][qy]
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) t[az * P1 + qy] = lds[(az * P1 + qy) * P1 + w][lane];
  // 4. z-pass -> u[qz][qy]
  T u[NP];
  cell_pass_z<T, P1, EO>(cf, t, u);
  // 5. quadrature-point terms: potential + y/z kinetic
  const int qx = w;
  const T kx = cf.kappa * cf.w[qx];
  const T* wv = P.wv + ee * (NP * P1);
  cell_point_terms<T, P1, EO>(cf, u, t, [&](int qz, int qy) { return wv[(qz * P1 + qy) * P1 + qx]; }, kx);
  // 6. t' = (B^T)_y (B^T)_z t  -> indexed [az][ay]
  T tp[NP];
  cell_back_yz<T, P1, EO>(cf, t, v, tp);
  // 7. s = kappa (B^T W)_y (B^T W)_z u  (the x kinetic term before its x-pass)
  cell_xkin_yz<T, P1, EO>(cf, u, v);
  // 8. transpose t' back to z-planes, x-pass with B^T
  __syncthreads();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) lds[(az * P1 + ay) * P1 + w][lane] = tp[az * P1 + ay];
  __syncthreads();
  T y[NP];
#pragma unroll
  for (int ay = 0; ay < P1; ++ay) {
    T r[P1];
#pragma unroll
    for (int q = 0; q < P1; ++q) r[q] = lds[(w * P1 + ay) * P1 + q][lane];
    cell_back_x<T, P1, EO>(cf, r, y + ay * P1);
  }
  // 9. transpose s, x-pass with B^T L1, accumulate
  __syncthreads();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) lds[(az * P1 + ay) * P1 + w][lane] = u[az * P1 + ay];
  __syncthreads();
#pragma unroll
  for (int ay = 0; ay < P1; ++ay) {
    T r[P1];
#pragma unroll
    for (int q = 0; q < P1; ++q) r[q] = lds[(w * P1 + ay) * P1 + q][lane];
#pragma unroll
    for (int ax = 0; ax < P1; ++ax) {
      T s = 0;
#pragma unroll
      for (int q = 0; q < P1; ++q) s += cf.BtL[ax][q] * r[q];
      y[ay * P1 + ax] += s;
    }
  }
  // 10. store plane az = w of y_e into the node-slot grid: local node a of cell c
  //     goes to slot (c (p+1) + a + 1) mod S per dimension, S = nc (p+1)
  if (valid) {
    const int S = nc * P1;
    int sz = cz * P1 + w + 1;
    if (sz >= S) sz -= S;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int sy = cy * P1 + ay + 1;
      if (sy >= S) sy -= S;
      const int64_t rowyz = (int64_t)S * (sy + (int64_t)S * sz);
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int sx = cx * P1 + ax + 1;
        if (sx >= S) sx -= S;
        Yc[(rowyz + sx) * ldc + j] = y[ay * P1 + ax];
      }
    }
  }
}

// Cell kernel with the planes in the lanes of one wave: lane = r * CWc + g holds plane r of
// the cell tensor for column g of a CWc-column block (CWc = 64 / P1 rounded down to even;
// the 64 - P1 CWc spare lanes repeat the last plane's work and store nothing).  A wave
// owns one (cell, column block) and its own LDS region, so the three transposes need no
// workgroup barrier and the four waves of a workgroup carry equal work.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The three products of small_gemm modes 1, 2 and 3 in one launch: every product is
// (n x n) times (n x columns), so one workgroup per block of kChainCols columns computes
//   W' = (sum of the folded tile partials) + H^oo Z^O,
//   out^O = alpha (S W' - c x^O) - beta prev^O,
//   Z^O of the next step = S out^O (when next),
// with S, H^oo and the block's Z^O, W' and out^O in LDS (1024 threads: one output of a phase
// per thread for n kChainCols <= 1024).  Sums run in the same order as in
// small_gemm (chunk partials first, then the products in k order); the chunk partials are
// loaded in batches of 8.
//
// Blocks of kChainColsCell columns and 256 threads run it as the first blocks of the cell launch, which
// it does not depend on, where a step is short (chain_in_cell): the same sums in the same order.
constexpr int kChainCols = 16;

constexpr int kChainColsCell = 4;
constexpr int64_t kChainInCellElems = (int64_t)1 << 23;  // most real elements of the step's blocks (chain_in_cell)

template <typename T, bool CPLX>
constexpr size_t enr_chain_lds_bytes(int n, int cols = kChainCols) {
  return (2 * (size_t)n * n + 3 * (size_t)n * cols) * (CPLX ? 2 : 1) * sizeof(T);
}

// fn_pptr null: the partials are folded (part2); else every function's are folded here
struct ChainArgs {
  int64_t N;
  int n, next;
  const int32_t *fn_pptr, *fn_poff;
  int nblk;      // leading blocks of a cell launch that run the chain, 0: none
  bool zo_only;  // they form Z^O = S x^O instead
};

// Z^O = S x^O by the first blocks of a cell launch (a thread per entry, sums in k order): a step outside a
// recurrence needs it at its node stage only
template <typename T, bool CPLX>
__device__ __forceinline__ void enr_zo(const KBatch<T>& kb, const ChainArgs& ca, int block) {
  constexpr int E = CPLX ? 2 : 1;
  const KP<T>& P = kb.k[blockIdx.z];
  const int m = P.nv, n = ca.n, t = block * 256 + (int)threadIdx.x, i = t / m, j = t - i * m;
  if (i >= n) return;
  const T* __restrict__ a = P.S + (int64_t)i * n * E;
  const T* __restrict__ b = P.x + ca.N * P.ldx + (int64_t)j * E;
  T sr = 0, si = 0;
#pragma unroll 8
  for (int k = 0; k < n; ++k) {
    if constexpr (!CPLX) {
      sr += a[k] * b[(int64_t)k * P.ldx];
    } else {
      const C2<T> q = cmul(C2<T>{a[2 * k], a[2 * k + 1]}, C2<T>{b[(int64_t)k * P.ldx], b[(int64_t)k * P.ldx + 1]});
      sr += q.r;
      si += q.i;
    }
  }
  P.zo[(int64_t)i * P.ncr + (int64_t)j * E] = sr;
  if (CPLX) P.zo[(int64_t)i * P.ncr + (int64_t)j * E + 1] = si;
}

template <typename T, bool CPLX, int TC>
__device__ __forceinline__ void enr_chain(const KBatch<T>& kb, const ChainArgs& ca, int block, unsigned char* chain_raw) {
  constexpr int E = CPLX ? 2 : 1;
  const int64_t N = ca.N;
  const int n = ca.n, next = ca.next;
  const int32_t* __restrict__ fn_pptr = ca.fn_pptr;
  const int32_t* __restrict__ fn_poff = ca.fn_poff;
  T* Ss = reinterpret_cast<T*>(chain_raw);  // [n][n] S
  T* Hs = Ss + (size_t)n * n * E;           // [n][n] H^oo
  T* Zs = Hs + (size_t)n * n * E;           // [n][TC] Z^O of this step
  T* Ws = Zs + (size_t)n * TC * E;          // [n][TC] W'
  T* Os = Ws + (size_t)n * TC * E;          // [n][TC] out^O
  const KP<T>& P = kb.k[blockIdx.z];
  const int m = P.nv, ncr = P.ncr;
  const int j0 = block * TC;
  if (j0 >= m) return;
  const int tid = threadIdx.x, nth = blockDim.x;
  for (int t = tid; t < n * n * E; t += nth) {
    Ss[t] = P.S[t];
    Hs[t] = P.Hoo[t];
  }
  for (int t = tid; t < n * TC; t += nth) {
    const int i = t / TC, jl = t - i * TC, j = min(j0 + jl, m - 1);
#pragma unroll
    for (int e = 0; e < E; ++e) Zs[(size_t)t * E + e] = P.zo[(int64_t)i * ncr + (int64_t)j * E + e];
  }
  __syncthreads();
  // sum_k A[i][k] B[k][jl] over LDS tiles, in k order
  auto dot = [&](const T* A, const T* B, int i, int jl, T& sr, T& si) {
    sr = 0;
    si = 0;
#pragma unroll 8
    for (int k = 0; k < n; ++k) {
      const T* a = A + ((size_t)i * n + k) * E;
      const T* b = B + ((size_t)k * TC + jl) * E;
      if constexpr (!CPLX) {
        sr += a[0] * b[0];
      } else {
        const C2<T> q = cmul(C2<T>{a[0], a[1]}, C2<T>{b[0], b[1]});
        sr += q.r;
        si += q.i;
      }
    }
  };
  // W'
  if (fn_pptr) {
    // every function has at most kReduceChunk partials: folded here, in the order of enr_reduce1_kernel
    for (int t = tid; t < n * TC; t += nth) {
      const int i = t / TC, jl = t - i * TC, j = min(j0 + jl, m - 1);
      // entry e of the list: group e mod 4, its even or odd entries; 8 entries at a time, their loads together
      // and the next positions beside them.  One by one, each entry is two dependent loads: with 27 partials of
      // each of 40 functions an application to 16 vectors takes 39.7 us so, 29.9 in batches.
      const int e0 = fn_pptr[i], cnt = fn_pptr[i + 1] - e0;
      const T* pj = P.part + (int64_t)j * E;
      T r[8] = {}, q[8] = {};
      int off[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) off[u] = cnt > 0 ? fn_poff[e0 + min(u, cnt - 1)] : 0;
      for (int e = 0; e < cnt; e += 8) {
        T v[8], w[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const T* p = pj + (int64_t)off[u] * ncr;
          v[u] = p[0];
          w[u] = CPLX ? p[E - 1] : T(0);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) off[u] = fn_poff[e0 + min(e + 8 + u, cnt - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u) {  // (an entry past the list is left out, not added as a product with 0)
          r[u] = e + u < cnt ? r[u] + v[u] : r[u];
          if (CPLX) q[u] = e + u < cnt ? q[u] + w[u] : q[u];
        }
      }
      T wr[4], wi[4];
#pragma unroll
      for (int grp = 0; grp < 4; ++grp) {
        wr[grp] = r[grp] + r[grp + 4];
        wi[grp] = q[grp] + q[grp + 4];
      }
      T sr, si;
      dot(Hs, Zs, i, jl, sr, si);
      Ws[(size_t)t * E] = ((wr[0] + wr[1]) + (wr[2] + wr[3])) + sr;
      if (CPLX) Ws[(size_t)t * E + 1] = ((wi[0] + wi[1]) + (wi[2] + wi[3])) + si;
    }
  } else if (m == 1) {
    // one column: the TC threads of a row, which would all compute the same entry, split its
    // chunks (thread jl adds chunks jl, jl + TC, ... in order) into Os, then add them in order
    for (int t = tid; t < n * TC; t += nth) {
      const int i = t / TC, jl = t - i * TC;
      const T* p2 = P.part2 + (int64_t)i * P.nch * ncr;
      T wr = 0, wi = 0;
      for (int ch = jl; ch < P.nch; ch += TC) {
        wr += p2[(int64_t)ch * ncr];
        if (CPLX) wi += p2[(int64_t)ch * ncr + 1];
      }
      Os[(size_t)t * E] = wr;
      if (CPLX) Os[(size_t)t * E + 1] = wi;
    }
    __syncthreads();
    for (int t = tid; t < n * TC; t += nth) {
      const int i = t / TC, jl = t - i * TC;
      T wr = 0, wi = 0;
      for (int q = 0; q < TC; ++q) {
        wr += Os[((size_t)i * TC + q) * E];
        if (CPLX) wi += Os[((size_t)i * TC + q) * E + 1];
      }
      T sr, si;
      dot(Hs, Zs, i, jl, sr, si);
      Ws[(size_t)t * E] = wr + sr;
      if (CPLX) Ws[(size_t)t * E + 1] = wi + si;
    }
  } else {
  for (int t = tid; t < n * TC; t += nth) {
    const int i = t / TC, jl = t - i * TC, j = min(j0 + jl, m - 1);
    const T* p2 = P.part2 + (int64_t)i * P.nch * ncr + (int64_t)j * E;
    T wr = 0, wi = 0;
    int ch = 0;
    for (; ch + 8 <= P.nch; ch += 8) {
      T vr[8], vi[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        vr[q] = p2[(int64_t)(ch + q) * ncr];
        vi[q] = CPLX ? p2[(int64_t)(ch + q) * ncr + 1] : T(0);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        wr += vr[q];
        if (CPLX) wi += vi[q];
      }
    }
    for (; ch < P.nch; ++ch) {
      wr += p2[(int64_t)ch * ncr];
      if (CPLX) wi += p2[(int64_t)ch * ncr + 1];
    }
    T sr, si;
    dot(Hs, Zs, i, jl, sr, si);
    Ws[(size_t)t * E] = wr + sr;
    if (CPLX) Ws[(size_t)t * E + 1] = wi + si;
  }
  }
  __syncthreads();
  // out^O
  for (int t = tid; t < n * TC; t += nth) {
    const int i = t / TC, jl = t - i * TC, j = j0 + jl;
    T sr, si;
    dot(Ss, Ws, i, jl, sr, si);
    const int64_t ox = (N + i) * P.ldx + (int64_t)min(j, m - 1) * E, oo = (N + i) * P.ldo + (int64_t)min(j, m - 1) * E;
    T alpha, cst, beta;
    step_scalars(P, alpha, cst, beta);
    T r = alpha * (sr - cst * P.x[ox]);
    if (beta != T(0)) r -= beta * P.prev[oo];
    T r2 = 0;
    if (CPLX) {
      r2 = alpha * (si - cst * P.x[ox + 1]);
      if (beta != T(0)) r2 -= beta * P.prev[oo + 1];
    }
    Os[(size_t)t * E] = r;
    if (CPLX) Os[(size_t)t * E + 1] = r2;
    if (j < m) {
      P.out[oo] = r;
      if (CPLX) P.out[oo + 1] = r2;
    }
  }
  if (!next) return;
  __syncthreads();
  // Z^O of the next step
  for (int t = tid; t < n * TC; t += nth) {
    const int i = t / TC, jl = t - i * TC, j = j0 + jl;
    T sr, si;
    dot(Ss, Os, i, jl, sr, si);
    if (j < m) {
      P.zn[(int64_t)i * ncr + (int64_t)j * E] = sr;
      if (CPLX) P.zn[(int64_t)i * ncr + (int64_t)j * E + 1] = si;
    }
  }
}

template <int P1>
constexpr int lanes_cw() { return (64 / P1) & ~1; }
template <typename T, int P1>
constexpr size_t cell_lanes_lds_bytes() { return 4 * (P1 * P1 * P1 * lanes_cw<P1>() + 128) * sizeof(T); }

// UF: the periodic-function k-point form's first-derivative term -i k . int N grad N is added
// (complex columns only): k . grad u at the Gauss points (derivatives of the interpolant of the
// Gauss values, the x-derivative taken on the x-y plane before the transpose), weighted, from
// the complex partner lane (real <-> imaginary part) with the sign of -i, into the values that
// the backward passes project.
//
// FIRST: what the launch's first ca.nblk blocks do instead.  An instance of its own each: the registers of the
// enrichment chain would be those of every cell block (complex128 degree 2: 64 without it, 124 with it).
enum class CellFirst { none, zo, chain };
// Whether the LDS is static, of a size the compiler knows: it then fits the registers to the waves that fit.  Not
// with a chain (its size), and not in float64 where that costs more than it gives: degree 3 would take 107
// registers with scalar ones spilled, four waves either way (an application to 90 vectors, 12^3 cells, 101 us so
// and 94 with 128), degree 4 with Z^O 167 for 157, three waves (band energy of 72 vectors 724 us and 722).
template <typename T, int P1, bool UF>
constexpr bool cell_lanes_own_lds(CellFirst first) {
  return first != CellFirst::chain &&
         !(sizeof(T) == 8 && !UF && (P1 == 4 || (P1 == 5 && first == CellFirst::zo)));
}
template <typename T, int P1, bool CPLX, bool UF, CellFirst FIRST>
__global__ __launch_bounds__(256, 3) void fe_cell_lanes_kernel(KBatch<T> kb, CellCoef<T> cf, int nc, int p, int n,
                                                            int64_t n_cells, int nch, ChainArgs ca) {
  static_assert(!UF || CPLX, "the first-derivative term acts on complex columns");
  constexpr int NP = P1 * P1;
  constexpr int CWc = lanes_cw<P1>();
  // degree 4: the even-odd passes (the periodic-function form, which runs in this kernel only,
  // keeps the plain sums in float64: there its first-derivative term needs the registers)
  constexpr bool EO = P1 == 5 && (!UF || sizeof(T) == 4);
  // launch order: the column chunks of a group of 4 cells are consecutive in L, and each
  // XCD (workgroups bk = x mod 8) takes a contiguous range of L, so that the chunks reading
  // the same node rows, and neighbouring cells, share one L2
  extern __shared__ __align__(16) unsigned char cell_raw[];
  if (FIRST != CellFirst::none && (int)blockIdx.x < ca.nblk) {  // the enrichment chain of this step, or its Z^O
    if constexpr (FIRST == CellFirst::zo) enr_zo<T, CPLX>(kb, ca, (int)blockIdx.x);
    if constexpr (FIRST == CellFirst::chain) enr_chain<T, CPLX, kChainColsCell>(kb, ca, (int)blockIdx.x, cell_raw);
    return;
  }
  const int nfirst = FIRST == CellFirst::none ? 0 : ca.nblk;
  const int nbk = (int)gridDim.x - nfirst, bk = (int)blockIdx.x - nfirst, nb8 = nbk & ~7;
  const int L = bk < nb8 ? (bk & 7) * (nb8 >> 3) + (bk >> 3) : bk;
  const int chunk = L % nch, cgrp = L / nch;
  constexpr bool own = cell_lanes_own_lds<T, P1, UF>(FIRST);
  __shared__ T lds_own[own ? 4 : 1][own ? NP * P1 * CWc : 1], wv_own[own ? 4 : 1][own ? 128 : 1];
  T(*lds_all)[NP * P1 * CWc] = reinterpret_cast<T(*)[NP * P1 * CWc]>(own ? (void*)lds_own : (void*)cell_raw);
  // W V of the wave's cell at its quadrature points
  T(*wv_all)[128] = reinterpret_cast<T(*)[128]>(own ? (void*)wv_own : (void*)(cell_raw + 4 * sizeof(lds_all[0])));
  const KP<T>& P = kb.k[blockIdx.z];
  const int ncr = P.ncr;
  if (chunk * CWc >= ncr) return;  // column block beyond this operator's width
  const T* __restrict__ X = P.x;
  const int64_t ldx = P.ldx;
  T* __restrict__ Yc = P.ycell;
  const int ldc = P.ldc;
  const Phase3<T> ph = P.ph;
  const int lane = threadIdx.x & 63;
  const int wid = threadIdx.x >> 6;
  const bool active = lane < P1 * CWc;
  const int w = min(lane / CWc, P1 - 1);  // plane of this lane
  const int g = active ? lane % CWc : lane - P1 * CWc;  // spare lanes repeat a last-plane lane
  T* lds = lds_all[wid];
  const int64_t e = (int64_t)cgrp * 4 + wid;
  const int j = chunk * CWc + g;
  const bool valid = (e < n_cells) && (j < ncr);
  // the wave's cell (uniform: scalar arithmetic); a wave past the last cell addresses the last
  // cell's nodes and stores nothing
  const int eu = (int)(e < n_cells ? e : n_cells - 1);  // n_cells < 2^31
  const int cx = eu % nc, cy = (eu / nc) % nc, cz = eu / (nc * nc);
  // W V of the wave's cell: loaded now, parked in LDS after the first passes, read in step 5
  constexpr int NQ3 = NP * P1;
  const T* __restrict__ wvg = P.wv + (e < n_cells ? e : n_cells - 1) * NQ3;
  const T wv0 = wvg[min(lane, NQ3 - 1)], wv1 = wvg[min(lane + 64, NQ3 - 1)];

  // 1. gather plane az = w with the m^-1/2 pre-scale (and Bloch phase)
  const int jc = min(j, ncr - 1);
  const T vmask = valid ? T(1) : T(0);
  T v[NP];
  {
    const int az = w;
    int iz = cz * p + az;
    bool wz = iz >= n;
    if (wz) iz -= n;
    // addresses: one 64-bit base per lane for its z-plane, then 32-bit row offsets from
    // full-rate 24-bit products (iy n ldx + ix ldx < n^2 ldx < 2^31, checked at launch)
    const T* __restrict__ Xz = X + (int64_t)iz * n * n * ldx + (CPLX ? (jc & ~1) : jc);
    const unsigned ldx32 = (unsigned)ldx, ldxn = (unsigned)ldx * (unsigned)n;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int iy = cy * p + ay;
      bool wy = iy >= n;
      if (wy) iy -= n;
      const unsigned oy = __umul24((unsigned)iy, ldxn);
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int ix = cx * p + ax;
        bool wx = ix >= n;
        if (wx) ix -= n;
        const unsigned off = oy + __umul24((unsigned)ix, ldx32);
        const T sc = cf.mscale * cf.om[ax] * cf.om[ay] * cf.om[az];
        // unconditional in-bounds loads (column clamped), zeroed by a multiply for lanes
        // outside the block: no branch around the load
        T val;
        if constexpr (!CPLX) {
          val = Xz[off];
        } else {
          const T* px = Xz + off;
          C2<T> z{px[0], px[1]};
          if (wx) z = cmul(z, C2<T>{ph.re[0], ph.im[0]});
          if (wy) z = cmul(z, C2<T>{ph.re[1], ph.im[1]});
          if (wz) z = cmul(z, C2<T>{ph.re[2], ph.im[2]});
          val = (jc & 1) ? z.i : z.r;
        }
        v[ay * P1 + ax] = sc * (val * vmask);
      }
    }
  }
  // 2. x- then y-pass with B1 (in registers)
  T t[NP];
  cell_pass_xy<T, P1, EO>(cf, v, t);
  // UF: x-derivative of the x-y plane (transposed after step 3, z-interpolated after step 4)
  T dxv[UF ? NP : 1];
  if constexpr (UF) {
#pragma unroll
    for (int qy = 0; qy < P1; ++qy)
#pragma unroll
      for (int qx = 0; qx < P1; ++qx) {
        T s = 0;
#pragma unroll
        for (int k = 0; k < P1; ++k) s += cf.Dh[qx][k] * v[qy * P1 + k];
        dxv[qy * P1 + qx] = s;
      }
  }
  // 3. transpose z-planes -> x-planes: lds[(az*P1 + qy)*P1 + qx]
  T* wvs = wv_all[wid];
  if (lane < NQ3) wvs[lane] = wv0;
  if (lane + 64 < NQ3) wvs[lane + 64] = wv1;
#pragma unroll
  for (int qy = 0; qy < P1; ++qy)
#pragma unroll
    for (int qx = 0; qx < P1; ++qx) lds[((w * P1 + qy) * P1 + qx) * CWc + g] = v[qy * P1 + qx];
  wave_sync();
  // this wave now owns qx = w; u[az][qy]
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) t[az * P1 + qy] = lds[((az * P1 + qy) * P1 + w) * CWc + g];
  if constexpr (UF) {
    wave_sync();  // every lane has read the transpose
#pragma unroll
    for (int qy = 0; qy < P1; ++qy)
#pragma unroll
      for (int qx = 0; qx < P1; ++qx) lds[((w * P1 + qy) * P1 + qx) * CWc + g] = dxv[qy * P1 + qx];
    wave_sync();
  }
  // 4. z-pass -> u[qz][qy]
  T u[NP];
  cell_pass_z<T, P1, EO>(cf, t, u);
  // UF: t = W' uk . grad u at this lane's Gauss points (W' the product of the 1D weights; t is
  // free after step 4), taken from the complex partner with the sign of -i: real part
  // += (k.G) imag, imag -= (k.G) real; the x-derivative read from the transposed plane in LDS
  if constexpr (UF) {
    const T k0 = P.uk[0], k1 = P.uk[1], k2 = P.uk[2];
    const T sg = (g & 1) ? T(-1) : T(1);
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) {
      T dt[P1];
#pragma unroll
      for (int k = 0; k < P1; ++k) dt[k] = lds[((k * P1 + qy) * P1 + w) * CWc + g];
#pragma unroll
      for (int qz = 0; qz < P1; ++qz) {
        T dx = 0, dy = 0, dz = 0;
#pragma unroll
        for (int k = 0; k < P1; ++k) {
          dx += cf.B1[qz][k] * dt[k];
          dy += cf.Dh[qy][k] * u[qz * P1 + k];
          dz += cf.Dh[qz][k] * u[k * P1 + qy];
        }
        const T tg = cf.w[w] * cf.w[qy] * cf.w[qz] * (k0 * dx + k1 * dy + k2 * dz);
        t[qz * P1 + qy] = sg * __shfl_xor(tg, 1);
      }
    }
  }
  // 5. quadrature-point terms: potential + y/z kinetic
  const int qx = w;
  const T kx = cf.kappa * cf.w[qx];
  if constexpr (UF) {
#pragma unroll
    for (int qz = 0; qz < P1; ++qz)
#pragma unroll
      for (int qy = 0; qy < P1; ++qy) {
        T ly = 0, lz = 0;
#pragma unroll
        for (int k = 0; k < P1; ++k) {
          ly += cf.L1[qy][k] * u[qz * P1 + k];
          lz += cf.L1[qz][k] * u[k * P1 + qy];
        }
        const T tq = wvs[(qz * P1 + qy) * P1 + qx] * u[qz * P1 + qy] + kx * (cf.w[qz] * ly + cf.w[qy] * lz);
        t[qz * P1 + qy] = tq + t[qz * P1 + qy];
      }
  } else {
    cell_point_terms<T, P1, EO>(cf, u, t, [&](int qz, int qy) { return wvs[(qz * P1 + qy) * P1 + qx]; }, kx);
  }
  // 6. t' = (B^T)_y (B^T)_z t  -> indexed [az][ay]
  T tp[NP];
  cell_back_yz<T, P1, EO>(cf, t, v, tp);
  // 7. s = kappa (B^T W)_y (B^T W)_z u  (the x kinetic term before its x-pass)
  cell_xkin_yz<T, P1, EO>(cf, u, v);
  // 8. transpose t' back to z-planes, x-pass with B^T
  wave_sync();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) lds[((az * P1 + ay) * P1 + w) * CWc + g] = tp[az * P1 + ay];
  wave_sync();
  T y[NP];
#pragma unroll
  for (int ay = 0; ay < P1; ++ay) {
    T r[P1];
#pragma unroll
    for (int q = 0; q < P1; ++q) r[q] = lds[((w * P1 + ay) * P1 + q) * CWc + g];
    cell_back_x<T, P1, EO>(cf, r, y + ay * P1);
  }
  // 9. transpose s, x-pass with B^T L1, accumulate
  wave_sync();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) lds[((az * P1 + ay) * P1 + w) * CWc + g] = u[az * P1 + ay];
  wave_sync();
#pragma unroll
  for (int ay = 0; ay < P1; ++ay) {
    T r[P1];
#pragma unroll
    for (int q = 0; q < P1; ++q) r[q] = lds[((w * P1 + ay) * P1 + q) * CWc + g];
#pragma unroll
    for (int ax = 0; ax < P1; ++ax) {
      T s = 0;
#pragma unroll
      for (int q = 0; q < P1; ++q) s += cf.BtL[ax][q] * r[q];
      y[ay * P1 + ax] += s;
    }
  }
  // 10. store plane az = w of y_e into the node-slot grid: local node a of cell c
  //     goes to slot (c (p+1) + a + 1) mod S per dimension, S = nc (p+1)
  if (valid && active) {
    const int S = nc * P1;
    int sz = cz * P1 + w + 1;
    if (sz >= S) sz -= S;
    // one 64-bit base per lane for its slot plane, 32-bit offsets below S^2 ldc < 2^31
    T* __restrict__ Ycz = Yc + (int64_t)sz * S * S * ldc + j;
    const unsigned ldc32 = (unsigned)ldc, ldcs = (unsigned)ldc * (unsigned)S;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int sy = cy * P1 + ay + 1;
      if (sy >= S) sy -= S;
      const unsigned oy = __umul24((unsigned)sy, ldcs);
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int sx = cx * P1 + ax + 1;
        if (sx >= S) sx -= S;
        Ycz[oy + __umul24((unsigned)sx, ldc32)] = y[ay * P1 + ax];
      }
    }
  }
}

// Cell stage at one real column (the auxiliary potential's conjugate gradients, Lanczos): the
// planes-in-lanes kernel with cells in the place of columns, lane = plane x CWc + cell of the
// wave, where the column layout would leave 11 of its 12 lane groups idle.  Every lane forms its
// own cell's addresses (64-bit), reads W V of its cell's points from device memory, and runs the
// same passes in the same order, so each cell's values equal the column layout's bit for bit.
template <typename T, int P1>
__global__ __launch_bounds__(256, 3) void fe_cell_cells_kernel(KBatch<T> kb, CellCoef<T> cf, int nc, int p, int n,
                                                               int64_t n_cells, ChainArgs ca) {
  constexpr int NP = P1 * P1;
  constexpr int CWc = lanes_cw<P1>();
  constexpr bool EO = P1 == 5;
  __shared__ T lds_all[4][NP * P1 * CWc];
  const KP<T>& P = kb.k[blockIdx.z];
  const T* __restrict__ X = P.x;
  const int64_t ldx = P.ldx, ldc = P.ldc;
  T* __restrict__ Yc = P.ycell;
  if ((int)blockIdx.x < ca.nblk) {
    enr_zo<T, false>(kb, ca, (int)blockIdx.x);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int wid = threadIdx.x >> 6;
  const bool active = lane < P1 * CWc;
  const int w = min(lane / CWc, P1 - 1);                // plane of this lane
  const int g = active ? lane % CWc : lane - P1 * CWc;  // cell of the wave; spare lanes repeat a last-plane lane
  T* lds = lds_all[wid];
  const int64_t e = ((int64_t)((int)blockIdx.x - ca.nblk) * 4 + wid) * CWc + g;
  const bool valid = e < n_cells;
  const int64_t eu = valid ? e : n_cells - 1;  // a lane past the last cell works on the last cell and stores nothing
  const int cx = (int)(eu % nc), cy = (int)((eu / nc) % nc), cz = (int)(eu / ((int64_t)nc * nc));
  const T vmask = valid ? T(1) : T(0);

  // 1. gather plane az = w with the m^-1/2 pre-scale
  T v[NP];
  {
    const int az = w;
    int iz = cz * p + az;
    if (iz >= n) iz -= n;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int iy = cy * p + ay;
      if (iy >= n) iy -= n;
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int ix = cx * p + ax;
        if (ix >= n) ix -= n;
        const T sc = cf.mscale * cf.om[ax] * cf.om[ay] * cf.om[az];
        const T val = X[(ix + (int64_t)n * (iy + (int64_t)n * iz)) * ldx];
        v[ay * P1 + ax] = sc * (val * vmask);
      }
    }
  }
  // 2. x- then y-pass
  T t[NP];
  cell_pass_xy<T, P1, EO>(cf, v, t);
  // 3. transpose z-planes -> x-planes
#pragma unroll
  for (int qy = 0; qy < P1; ++qy)
#pragma unroll
    for (int qx = 0; qx < P1; ++qx) lds[((w * P1 + qy) * P1 + qx) * CWc + g] = v[qy * P1 + qx];
  wave_sync();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) t[az * P1 + qy] = lds[((az * P1 + qy) * P1 + w) * CWc + g];
  // 4. z-pass
  T u[NP];
  cell_pass_z<T, P1, EO>(cf, t, u);
  // 5. quadrature-point terms (W V of this lane's cell at the points of its plane)
  const int qx = w;
  const T kx = cf.kappa * cf.w[qx];
  const T* __restrict__ wvc = P.wv + eu * (NP * P1);
  cell_point_terms<T, P1, EO>(cf, u, t, [&](int qz, int qy) { return wvc[(qz * P1 + qy) * P1 + qx]; }, kx);
  // 6. t' = (B^T)_y (B^T)_z t; 7. the x kinetic term before its x-pass
  T tp[NP];
  cell_back_yz<T, P1, EO>(cf, t, v, tp);
  cell_xkin_yz<T, P1, EO>(cf, u, v);
  // 8. transpose t' back to z-planes, x-pass with B^T
  wave_sync();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) lds[((az * P1 + ay) * P1 + w) * CWc + g] = tp[az * P1 + ay];
  wave_sync();
  T y[NP];
#pragma unroll
  for (int ay = 0; ay < P1; ++ay) {
    T r[P1];
#pragma unroll
    for (int q = 0; q < P1; ++q) r[q] = lds[((w * P1 + ay) * P1 + q) * CWc + g];
    cell_back_x<T, P1, EO>(cf, r, y + ay * P1);
  }
  // 9. transpose s, x-pass with B^T L1, accumulate
  wave_sync();
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) lds[((az * P1 + ay) * P1 + w) * CWc + g] = u[az * P1 + ay];
  wave_sync();
#pragma unroll
  for (int ay = 0; ay < P1; ++ay) {
    T r[P1];
#pragma unroll
    for (int q = 0; q < P1; ++q) r[q] = lds[((w * P1 + ay) * P1 + q) * CWc + g];
#pragma unroll
    for (int ax = 0; ax < P1; ++ax) {
      T s = 0;
#pragma unroll
      for (int q = 0; q < P1; ++q) s += cf.BtL[ax][q] * r[q];
      y[ay * P1 + ax] += s;
    }
  }
  // 10. store plane az = w of the cell's result into the node-slot grid (column 0)
  if (valid && active) {
    const int S = nc * P1;
    int sz = cz * P1 + w + 1;
    if (sz >= S) sz -= S;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int sy = cy * P1 + ay + 1;
      if (sy >= S) sy -= S;
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int sx = cx * P1 + ax + 1;
        if (sx >= S) sx -= S;
        Yc[(sx + (int64_t)S * (sy + (int64_t)S * sz)) * ldc] = y[ay * P1 + ax];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// BF16 cell kernel (real operators, float32 vectors): the cell operator in dense form
//   U = B Z,  T = (W V) o U,  Y = K Z + B^T T
// on the matrix cores (16x16x32 bf16 MFMA, float32 accumulation), with B, K, B^T
// (128 x 128, zero-padded) held in LDS in A-fragment order.  Z (nodes x 16 columns of
// one cell, m^-1/2 pre-scaled) and T are rounded to bf16; U and Y stay float32.  The
// lane layout of the result of B Z is the operand layout of B^T T up to a fixed
// permutation of each 32-point block, which is built into the stored B^T.  Each wave
// takes (cell, 16-column block) tasks in turn; Y goes to the node-slot grid.
// ---------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBf16MatElems = 8 * 4 * 64 * 8;  // one 128 x 128 matrix in fragment order

__global__ __launch_bounds__(768) void fe_cell_bf16_kernel(KBatch<float> kb, const uint16_t* __restrict__ mats,
                                                           CellCoef<float> cf, int nc, int p, int n, int P1,
                                                           int64_t n_cells) {
  extern __shared__ unsigned char smem_raw[];
  bf16x8* frag = reinterpret_cast<bf16x8*>(smem_raw);  // [3][8][4][64]
  // per local node a < 128: (ax, ay, az) packed in 8-bit fields, and the m^-1/2 factor
  int* ncode = reinterpret_cast<int*>(smem_raw + 3 * kBf16MatElems * sizeof(uint16_t));
  float* nscale = reinterpret_cast<float*>(ncode + 128);
  // offsets of local node a from the cell's first node (global rows) and first slot (grid
  // rows), valid for cells that do not touch the upper periodic boundary
  int* noff = reinterpret_cast<int*>(nscale + 128);
  int* soff = noff + 128;
  const int nd = P1 * P1 * P1;
  {
    const uint4* src = reinterpret_cast<const uint4*>(mats);
    uint4* dst = reinterpret_cast<uint4*>(smem_raw);
    for (int i = threadIdx.x; i < 3 * kBf16MatElems / 8; i += blockDim.x) dst[i] = src[i];
    if (threadIdx.x < 128) {
      const int a = threadIdx.x;
      const int ax = a % P1, ay = (a / P1) % P1, az = a / (P1 * P1);
      float om[kMaxP1];
#pragma unroll
      for (int i = 0; i < kMaxP1; ++i) om[i] = cf.om[i];
      float sx = 0.f, sy = 0.f, sz = 0.f;
#pragma unroll
      for (int i = 0; i < kMaxP1; ++i) {
        sx = i == ax ? om[i] : sx;
        sy = i == ay ? om[i] : sy;
        sz = i == az ? om[i] : sz;
      }
      ncode[a] = a < nd ? (ax | (ay << 8) | (az << 16)) : 0;
      nscale[a] = a < nd ? cf.mscale * sx * sy * sz : 0.0f;
      noff[a] = a < nd ? ax + n * (ay + n * az) : 0;
      soff[a] = a < nd ? ax + nc * P1 * (ay + nc * P1 * az) : 0;
    }
  }
  __syncthreads();
  const bf16x8* fB = frag;
  const bf16x8* fK = frag + kBf16MatElems / 8;
  const bf16x8* fBT = frag + 2 * kBf16MatElems / 8;
  const KP<float>& P = kb.k[blockIdx.z];
  const int ncr = P.ncr;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int c = lane & 15, g = lane >> 4;
  const int ncb = (ncr + 15) / 16;
  const int64_t ntask = n_cells * ncb;
  const float* __restrict__ X = P.x;
  const int64_t ldx = P.ldx;
  float* __restrict__ Yc = P.ycell;
  const int64_t ldc = P.ldc;
  const int S = nc * P1;
  // workgroups of one XCD (blockIdx.x = x mod 8) take a contiguous range of task groups,
  // so that the column blocks of a cell and neighbouring cells share one L2
  const int nbk = gridDim.x, bk = blockIdx.x, nb8 = nbk & ~7;
  const int wg = bk < nb8 ? (bk & 7) * (nb8 >> 3) + (bk >> 3) : bk;
  for (int64_t task = (int64_t)wg * nw + w; task < ntask; task += (int64_t)gridDim.x * nw) {
    const int64_t e = task / ncb;
    const int col = (int)(task - e * ncb) * 16 + c;
    const bool cok = col < ncr;
    const int cc = cok ? col : ncr - 1;
    const int cx = (int)(e % nc), cy = (int)((e / nc) % nc), cz = (int)(e / ((int64_t)nc * nc));
    const int bx = cx * p, by = cy * p, bz = cz * p;
    // Z: node 32 k4 + 8 g + t of the cell, column col, scaled by m^-1/2 (one batch of loads);
    // a cell away from the upper periodic boundary (wave-uniform) indexes by table offsets
    const bool interior = cx < nc - 1 && cy < nc - 1 && cz < nc - 1;
    const int64_t gbase = bx + (int64_t)n * (by + (int64_t)n * bz);
    // W V of this lane's quadrature points, loaded with the gather (used after U = B Z)
    const float* wv = P.wv + e * nd;
    float wq[4][8];
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int q0 = 32 * k4 + 4 * g + v, q1 = q0 + 16;
        wq[k4][v] = wv[q0 < nd ? q0 : 0];
        wq[k4][4 + v] = wv[q1 < nd ? q1 : 0];
      }
    bf16x8 z[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // two batches of 16 loads
      float zv[16];
      if (interior) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int a = 32 * (2 * h + (i >> 3)) + 8 * g + (i & 7);
          zv[i] = X[(gbase + noff[a]) * ldx + cc];
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int a = 32 * (2 * h + (i >> 3)) + 8 * g + (i & 7);
          const int code = ncode[a];
          int ix = bx + (code & 255), iy = by + ((code >> 8) & 255), iz = bz + (code >> 16);
          ix -= ix >= n ? n : 0;
          iy -= iy >= n ? n : 0;
          iz -= iz >= n ? n : 0;
          zv[i] = X[(ix + (int64_t)n * (iy + (int64_t)n * iz)) * ldx + cc];
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i)
        z[2 * h + (i >> 3)][i & 7] = (__bf16)(zv[i] * nscale[32 * (2 * h + (i >> 3)) + 8 * g + (i & 7)]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // U = B Z
    f32x4 u[8];
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      u[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4)
        u[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fB[(mb * 4 + k4) * 64 + lane], z[k4], u[mb], 0, 0, 0);
    }
    // T = (W V) o U, as the operand of B^T T (point 16 mb + 4 g + v of U sits in lane g, element v)
    bf16x8 tq[4];
#pragma unroll
    for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int q0 = 32 * k4 + 4 * g + v, q1 = q0 + 16;
        tq[k4][v] = (__bf16)(q0 < nd ? wq[k4][v] * u[2 * k4][v] : 0.0f);
        tq[k4][4 + v] = (__bf16)(q1 < nd ? wq[k4][4 + v] * u[2 * k4 + 1][v] : 0.0f);
      }
    // Y = K Z + B^T T, stored to the node-slot grid
#pragma unroll 2
    for (int mb = 0; mb < 8; ++mb) {
      f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4) {
        y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fK[(mb * 4 + k4) * 64 + lane], z[k4], y, 0, 0, 0);
        y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fBT[(mb * 4 + k4) * 64 + lane], tq[k4], y, 0, 0, 0);
      }
      if (interior) {
        const int64_t sbase = (cx * P1 + 1) + (int64_t)S * ((cy * P1 + 1) + (int64_t)S * (cz * P1 + 1));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * mb + 4 * g + v;
          if (cok && a < nd) Yc[(sbase + soff[a]) * ldc + col] = y[v];
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 16 * mb + 4 * g + v;
          if (cok && a < nd) {
            const int code = ncode[a];
            int sx = cx * P1 + (code & 255) + 1, sy = cy * P1 + ((code >> 8) & 255) + 1,
                sz = cz * P1 + (code >> 16) + 1;
            sx -= sx >= S ? S : 0;
            sy -= sy >= S ? S : 0;
            sz -= sz >= S ? S : 0;
            Yc[(sx + (int64_t)S * (sy + (int64_t)S * sz)) * ldc + col] = y[v];
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Node stage: out = alpha (m^-1/2 sum_slots(Y) + Ht_t Z^O - c x) - beta prev on the FE rows, and the
// tile's partial part_t = Ht_t^* X_t of the enrichment rows' H^co* X (Ht_t: the tile's dense block of
// m^-1/2 H^co).
//
// One wave per (half a coupling tile of kTileRows rows, column group of 16 NC real columns); the waves
// of up to 4 column groups share the tile's coupling block in LDS, copied there without passing
// through registers, and a table of what each row needs (offsets, factors, flags).  A wave holds its
// rows in the layout of the 16x16x4 MFMA result (row 16 rb + M::row(lane, v), column lane % 16), so that
// Ht_t Z^O, slot sums, X, previous iterate and output meet in registers without a transpose; the loads of X and
// of the first slot pairs are issued before the first is used, then those of the previous iterate (in float32
// behind them; in float64 the test for it is a value per lane to the compiler, so they wait for the earlier
// ones and go out one by one).  In a recurrence the partial is formed from the result,
// which is the next step's X: only there are rows exchanged (LDS tile of the column group), each half
// taking alternate blocks of 16 functions.
//
// What bounds it: memory latency against waves in flight.  At 128 registers 16 waves are resident on a
// CU (a kernel of 16 rows x 64 columns per wave, X and Z^O through LDS: 8).  diamond64, 320 columns:
// float64 3750 -> 3030 us (13.6 GB, 4.5 TB/s of the copy kernel's 5.5), float32 1870 -> 1470 us; diamond8,
// 72 columns: 110 -> 100 us and 54 -> 60 us (17 thousand waves: 4.2 rounds of the device); Bloch operators,
// four k-points of 67..96 complex128 columns: 1000 us beside the cell stage + 600 us in two kernels ->
// 1050 us in one (a degree 2000 -> 1690 us).
//
// Complex columns are interleaved (re, im); a complex product is two real MFMA passes over the real
// and imaginary parts of Ht with the matching (swapped, signed) columns.
// ---------------------------------------------------------------------------
template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
  typedef double V4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V4 op(double a, double b, V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of the 16x16 result held by lane l in element v (column l % 16)
  static __device__ __forceinline__ int row(int l, int v) { return (l >> 4) + 4 * v; }
};
template <>
struct Mfma<float> {
  typedef float V4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V4 op(float a, float b, V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int l, int v) { return 4 * (l >> 4) + v; }
};

// a / p for the supported element degrees p = 2, 3, 4 (a >= 0): constant divisors
__device__ __forceinline__ int div_p(int a, int p) { return p == 4 ? a >> 2 : (p == 2 ? a >> 1 : a / 3); }

constexpr int kNodeGroups = 4;  // column groups of a node workgroup at most: two waves each

// NC consecutive columns of a row, loaded or stored together (rows need not be aligned to pairs)
template <typename T, int NC>
struct ColVec {
  T e[NC];
};
template <typename T, int NC>
__device__ __forceinline__ ColVec<T, NC> load_cols(const T* p) {
  ColVec<T, NC> r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}

// LDS of a node workgroup whose waves work on up to ntl consecutive tiles: their coupling blocks as
// they are stored (one after the other, see tile_offset), in whole 1 KB pieces (one 16-byte element
// per lane) and with 16 functions to spare, read past the last row and unused; then their lists.
template <typename T, bool CPLX>
__host__ __device__ constexpr size_t node_block_bytes(int fpmax, int pad, int ntl) {
  return ((size_t)(kTileRows * (fpmax + pad) * ntl + 16) * (CPLX ? 2 : 1) * sizeof(T) + 1023) / 1024 * 1024;
}
__host__ __device__ constexpr size_t node_list_bytes(int fpmax, int ntl) {
  return ((size_t)ntl * fpmax + 63) / 64 * 64 * sizeof(int32_t);  // 64 entries (one per lane) at a time
}
// What the node stage needs of each tile row, formed once per workgroup: the FE row, element offset of its
// first slot in the node-slot grid, m^-1/2, the step to the next slot where the node is shared in x
// (else 0), flags (shared in y, z: a second slot there; first slot a periodic image in x, y, z; in
// the mesh).  Rows past the mesh: those of row 0, no flags.
template <typename T>
struct alignas(8) NodeRow {
  int64_t slot;
  T msc;
  int32_t row, dx, flags;
};
enum { kY2 = 1, kZ2 = 2, kXW = 4, kYW = 8, kZW = 16, kIn = 32 };
// Work space of a node workgroup: the blocks, the rows of its tiles, their lists, and a
// kTileRows x (16 NC) tile of values per column group
struct NodeLds {
  size_t rows, lists, x, total;
};
template <typename T, bool CPLX, int NC>
__host__ __device__ constexpr NodeLds node_lds(int fpmax, int pad, int ntl, int groups) {
  NodeLds l{};
  l.rows = fpmax > 0 ? node_block_bytes<T, CPLX>(fpmax, pad, ntl) : 0;
  l.lists = l.rows + (size_t)ntl * kTileRows * sizeof(NodeRow<T>);
  l.x = l.lists + node_list_bytes(fpmax, ntl);
  l.total = l.x + (fpmax > 0 ? (size_t)groups * kTileRows * 16 * NC * sizeof(T) : 0);
  return l;
}
// tiles that w consecutive (tile, column group) items touch, the first at a multiple of w, gp
// groups per tile
__host__ __device__ constexpr int node_tiles(int gp, int w) {
  return gp % w == 0 ? 1 : (w % gp == 0 ? w / gp : (w - 1 + gp - 1) / gp + 1);
}

// A wave's share of the node stage: half the rows of a tile (two groups of 16) x a column group, and the
// tile's coupling block and list in LDS.
struct NodeItem {
  int t, dt, cb0, f0, FP;  // tile, and its place among the workgroup's
  size_t blk;  // byte offset of the tile's block in LDS
  int list;    // first entry of its list
  int half, grp;  // which half of the tile; column group of the workgroup
  bool live;   // else the wave only helps with the copies
};

// The mesh of a node or part kernel launch
struct NodeMesh {
  int nc, p, n, P1, N, tm, ntiles;
  int fpmax, pad, ntl, span;
};

// span: a workgroup's waves take consecutive (tile, column group) items across tile ends; else each
// tile's groups are padded to whole workgroups.  Launch order: the column groups of a tile are
// consecutive, and each XCD (workgroups bk = x mod 8) takes a contiguous range, so the groups that
// read the same coupling block, and neighbouring tiles, share one L2.  Starts the copies of the blocks
// and lists and forms the rows (cf not null); both are to be followed by a barrier.  Returns false (the
// whole workgroup) past the operator's items.
template <typename T, bool CPLX, int NC>
__device__ __forceinline__ bool node_item(const KP<T>& P, const NodeMesh& g, const int32_t* __restrict__ tile_fptr,
                                          const int32_t* __restrict__ tile_fns, const CellCoef<T>* cf,
                                          unsigned char* smem, const NodeLds& lds, NodeItem& it) {
  constexpr int E = CPLX ? 2 : 1;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), nw = (int)(blockDim.x >> 6), W = nw >> 1;
  it.half = w & 1;
  it.grp = w >> 1;
  const int G = (P.ncr + 16 * NC - 1) / (16 * NC), GP = g.span ? G : (G + W - 1) / W * W;  // groups of a tile
  const int items = g.ntiles * GP, nbk = (items + W - 1) / W, bk = blockIdx.x, nb8 = nbk & ~7;
  if (bk >= nbk) return false;
  const int L = bk < nb8 ? (bk & 7) * (nb8 >> 3) + (bk >> 3) : bk;
  const int item = min(L * W + it.grp, items - 1);
  const int t0 = L * W / GP, t1 = min(L * W + W - 1, items - 1) / GP;  // the workgroup's tiles
  it.t = item / GP;
  it.dt = it.t - t0;
  it.cb0 = (item - it.t * GP) * 16 * NC;
  it.live = L * W + it.grp < items && it.cb0 < P.ncr;
  if (!it.live) it.cb0 = 0;  // its loads stay in bounds, it stores nothing
  it.f0 = it.FP = it.list = 0;
  it.blk = 0;
  if (tile_fptr) {
    const int fa = tile_fptr[t0], fb = tile_fptr[t1 + 1];
    it.f0 = tile_fptr[it.t];
    it.FP = tile_fptr[it.t + 1] - it.f0;
    it.list = it.f0 - fa;
    it.blk = (size_t)(tile_offset(it.f0, it.t, g.pad) - tile_offset(fa, t0, g.pad)) * E * sizeof(T);
    const unsigned char* src = reinterpret_cast<const unsigned char*>(P.tv + tile_offset(fa, t0, g.pad) * E);
    const unsigned nbytes = (unsigned)((tile_offset(fb, t1 + 1, g.pad) - tile_offset(fa, t0, g.pad)) * E * sizeof(T));  // 256 m
    for (unsigned q = (unsigned)w * 1024u; q < nbytes; q += (unsigned)nw * 1024u) {
      const unsigned o = min(q + (unsigned)lane * 16u, nbytes - 16u);  // the last piece: in bounds, not used
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + o),
                                       (__attribute__((address_space(3))) void*)(smem + q), 16, 0, 0);
    }
    for (int q = w * 64; q < fb - fa; q += nw * 64)  // the lists, 64 entries a wave
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(tile_fns + min(fa + q + lane, fb - 1)),
          (__attribute__((address_space(3))) void*)(smem + lds.lists + (size_t)q * sizeof(int32_t)), 4, 0, 0);
  }
  if (cf) {
    NodeRow<T>* rows = reinterpret_cast<NodeRow<T>*>(smem + lds.rows);
    const int S = g.nc * g.P1;
    for (int q = threadIdx.x; q < (t1 - t0 + 1) * kTileRows; q += blockDim.x) {
      int x0, y0, z0, ix, iy, iz;
      tile_origin(t0 + q / kTileRows, g.n, g.tm, x0, y0, z0);
      const bool in = tile_row_coords(x0, y0, z0, q % kTileRows, g.n, g.tm, ix, iy, iz) >= 0;
      // slots of node i per dimension: a shared node (i mod p == 0) has two, the one from the lower
      // cell first; slot 0 holds the periodic image of the last cell
      const int qx = div_p(ix, g.p), rx = ix - qx * g.p, qy = div_p(iy, g.p), ry = iy - qy * g.p,
                qz = div_p(iz, g.p), rz = iz - qz * g.p;
      const int bx = qx * g.P1 + (rx ? rx + 1 : 0), by = qy * g.P1 + (ry ? ry + 1 : 0),
                bz = qz * g.P1 + (rz ? rz + 1 : 0);
      NodeRow<T> r;
      r.row = in ? ix + g.n * (iy + g.n * iz) : 0;
      r.slot = in ? slot_index(bx, by, bz, S) * P.ldc : 0;
      r.msc = cf->mscale * cf->om[rx] * cf->om[ry] * cf->om[rz];
      r.dx = in && rx == 0 ? P.ldc : 0;
      r.flags = in ? kIn | (ry == 0 ? kY2 : 0) | (rz == 0 ? kZ2 : 0) | (bx == 0 ? kXW : 0) | (by == 0 ? kYW : 0) |
                         (bz == 0 ? kZW : 0)
                   : 0;
      rows[q] = r;
    }
  }
  return true;
}

// Barrier of the workgroup for LDS written by its waves; loads from memory stay under way
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// Barrier for the blocks and lists copied by node_item, without waiting for the loads issued after v: a
// wave's copies were issued before the load of v and loads complete in order, so they are in LDS once v is
// here.  v has to be the loaded value itself, of a load that every wave issues: behind a select the compiler
// may turn the load into a branch around it, and a wave without an active lane there would wait for nothing.
template <typename V>
__device__ __forceinline__ void copied_barrier(V v) {
  asm volatile("" ::"v"(v));
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The same, waiting for everything the wave has under way
__device__ __forceinline__ void copied_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// part_t[f][columns] = Ht_t^* X_t, in two parts: the two waves of a column group put their rows of X_t
// (x[rb][v], in the layout of the MFMA result; 0 past the mesh) into the group's LDS tile, then, after a
// barrier of the whole workgroup, take alternate blocks of 16 functions over all rows (functions past
// the list give rows that are not stored).
template <typename T, int NC>
__device__ __forceinline__ void node_stash(T* xt, const NodeItem& it, const ColVec<T, NC> (&x)[2][4]) {
  const int lane = threadIdx.x & 63;
  ColVec<T, NC>* xs = reinterpret_cast<ColVec<T, NC>*>(xt) + it.grp * kTileRows * 16;  // [kTileRows][16]
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      xs[(it.half * 32 + rb * 16 + Mfma<T>::row(lane, v)) * 16 + (lane & 15)] = x[rb][v];
}
template <typename T, bool CPLX, int NC>
__device__ __forceinline__ void node_part(const KP<T>& P, const T* hs, int HS, const T* xt, const NodeItem& it) {
  using M = Mfma<T>;
  using V4 = typename M::V4;
  using CV = ColVec<T, NC>;
  constexpr int E = CPLX ? 2 : 1;
  const int lane = threadIdx.x & 63, li = lane & 15, FP = it.FP, ncr = P.ncr;
  const int col = it.cb0 + NC * li;
  const CV* xs = reinterpret_cast<const CV*>(xt) + it.grp * kTileRows * 16;
  lds_barrier();
  if (!it.live) return;
  const T sp = (li & 1) ? T(-1) : T(1);  // NC = 1: sign of the partner's part
  for (int m0 = 16 * it.half; m0 < FP; m0 += 32) {
    V4 pc[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) pc[j] = V4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < kTileRows / 4; ++ks) {
      const int r = 4 * ks + (lane >> 4);
      const T* h = hs + (unsigned)(r * HS + m0 + li) * E;
      const CV xv = xs[r * 16 + li];
      if constexpr (CPLX) {
        const T hr = h[0], hi = h[1];
#pragma unroll
        for (int j = 0; j < NC; ++j) pc[j] = M::op(hr, xv.e[j], pc[j]);
        if constexpr (NC == 2) {
          pc[0] = M::op(hi, xv.e[1], pc[0]);
          pc[1] = M::op(-hi, xv.e[0], pc[1]);
        } else {
          pc[0] = M::op(hi, sp * __shfl_xor(xv.e[0], 1), pc[0]);
        }
      } else {
        const T hv = h[0];
#pragma unroll
        for (int j = 0; j < NC; ++j) pc[j] = M::op(hv, xv.e[j], pc[j]);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int f = m0 + M::row(lane, v);
      T* o = P.part + (int64_t)(it.f0 + f) * ncr + col;
      if (f < FP) {
        if (NC == 2 && col + 1 < ncr) {
          const ColVec<T, 2> q{{pc[0][v], pc[NC - 1][v]}};
          __builtin_memcpy(o, &q, sizeof(q));
        } else if (col < ncr) {
          o[0] = pc[0][v];
        }
      }
    }
  }
}

// X of a wave's columns: from clamped columns (loads stay in bounds; the values of columns past ncr
// are not used).  NC = 2 needs ncr >= 2; an odd last column sits in the second element of the pair
// that ends there.
template <typename T, int NC>
__device__ __forceinline__ ColVec<T, NC> load_row(const T* row, int col, int ncr) {
  ColVec<T, NC> r = load_cols<T, NC>(row + min(col, ncr - NC));
  if constexpr (NC == 2) {
    if (ncr & 1) r.e[0] = col == ncr - 1 ? r.e[1] : r.e[0];
  }
  return r;
}

// part of a block's first step (later steps form it from their result): fe_part_kernel, same tiles
// and column groups as the node kernel
template <typename T, bool CPLX, int NC>
__global__ __launch_bounds__(128 * kNodeGroups, 4) void fe_part_kernel(KBatch<T> kb, NodeMesh g,
                                                                       const int32_t* __restrict__ tile_fptr,
                                                                       const int32_t* __restrict__ tile_fns) {
  using M = Mfma<T>;
  extern __shared__ unsigned char smem_raw[];
  const KP<T>& P = kb.k[blockIdx.z];
  const NodeLds lds = node_lds<T, CPLX, NC>(g.fpmax, g.pad, g.ntl, (int)(blockDim.x >> 7));
  NodeItem it;
  if (!node_item<T, CPLX, NC>(P, g, tile_fptr, tile_fns, nullptr, smem_raw, lds, it)) return;
  const int lane = threadIdx.x & 63, col = it.cb0 + NC * (lane & 15);
  int tx0, ty0, tz0;
  tile_origin(it.t, g.n, g.tm, tx0, ty0, tz0);
  ColVec<T, NC> x[2][4];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int gr = tile_row_node(tx0, ty0, tz0, it.half * 32 + rb * 16 + M::row(lane, v), g.n, g.tm);
      x[rb][v] = load_row<T, NC>(P.x + (int64_t)max(gr, 0) * P.ldx, col, P.ncr);
#pragma unroll
      for (int j = 0; j < NC; ++j) x[rb][v].e[j] = gr >= 0 ? x[rb][v].e[j] : T(0);
    }
  copied_barrier();  // (x went through selects: no value of it stands for the copies)
  T* xt = reinterpret_cast<T*>(smem_raw + lds.x);
  node_stash<T, NC>(xt, it, x);
  node_part<T, CPLX, NC>(P, reinterpret_cast<const T*>(smem_raw + it.blk), it.FP + g.pad, xt, it);
}

// PX: part of this step's X (a single application); else part of the step's result, which is the next
// step's X, when pnext.
template <typename T, bool CPLX, int NC, bool PX>
__global__ __launch_bounds__(128 * kNodeGroups, 4) void fe_node_kernel(KBatch<T> kb, NodeMesh g, CellCoef<T> cf,
                                                                       const int32_t* __restrict__ tile_fptr,
                                                                       const int32_t* __restrict__ tile_fns, int pnext) {
  using M = Mfma<T>;
  using V4 = typename M::V4;
  using CV = ColVec<T, NC>;
  constexpr int E = CPLX ? 2 : 1, RB = 2;  // groups of 16 rows of a wave
  extern __shared__ unsigned char smem_raw[];
  const KP<T>& P = kb.k[blockIdx.z];
  const int ncr = P.ncr;
  const NodeLds lds = node_lds<T, CPLX, NC>(g.fpmax, g.pad, g.ntl, (int)(blockDim.x >> 7));
  NodeItem it;
  if (!node_item<T, CPLX, NC>(P, g, tile_fptr, tile_fns, &cf, smem_raw, lds, it)) return;
  const int FP = it.FP, rb0 = 2 * it.half;  // the wave's rows: groups rb0, rb0 + 1 of the tile
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int col = it.cb0 + NC * li;
  const T* hs = reinterpret_cast<const T*>(smem_raw + it.blk);  // [kTileRows][HS][E]
  const int32_t* fs = reinterpret_cast<const int32_t*>(smem_raw + lds.lists) + it.list;
  const NodeRow<T>* rows = reinterpret_cast<const NodeRow<T>*>(smem_raw + lds.rows) + it.dt * kTileRows + rb0 * 16;
  T* xt = reinterpret_cast<T*>(smem_raw + lds.x);
  const int HS = FP + g.pad;
  T alpha, c, beta;
  step_scalars(P, alpha, c, beta);

  const int colx = min(col, ncr - NC);  // columns of the loads of X, Z^O and prev (see load_row)
  auto fix_odd = [&](CV& r) {
    if constexpr (NC == 2) {
      if (ncr & 1) r.e[0] = col == ncr - 1 ? r.e[1] : r.e[0];
    }
  };
  lds_barrier();  // the rows

  // ---- loads of all the wave's rows (element v of group rb: row 16 rb + M::row(lane, v)):
  // X; the first slot pair of every node, its lower-x slot and, where it is shared in x, the next one
  // (else the first again: in bounds, cached, discarded); the previous iterate (read before any element
  // of out, which may be the same array, is written).  Slot columns past ncr (ldc >= ncr) read the next
  // row or the grid's padding (slot_grid_elems)
  auto row = [&](int rb, int v) -> const NodeRow<T>& { return rows[rb * 16 + M::row(lane, v)]; };
  const T* __restrict__ Xc = P.x + colx;
  const T* __restrict__ Y = P.ycell + col;
  CV xr[RB][4], sa[RB][4], sb[RB][4], pv[RB][4];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) xr[rb][v] = load_cols<T, NC>(Xc + row(rb, v).row * P.ldx);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const T* ya = Y + row(rb, v).slot;
      sa[rb][v] = load_cols<T, NC>(ya);
      sb[rb][v] = load_cols<T, NC>(ya + row(rb, v).dx);
    }
  const bool use_prev = beta != T(0);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (use_prev) {
        pv[rb][v] = load_cols<T, NC>(P.prev + colx + row(rb, v).row * P.ldo);
      } else {
#pragma unroll
        for (int j = 0; j < NC; ++j) pv[rb][v].e[j] = T(0);
      }
    }
  if (tile_fptr) copied_barrier(xr[RB - 1][3].e[0]);

  // ---- node-slot sums: the lower-x slot a and (shared x node) the next one b of (ky, kz) pair kk, masks
  // as factors (the gathered values are finite)
  auto pair_sum = [&](int f, int dx, int kk, CV a, CV b) {
    const T m2 = dx ? T(1) : T(0);
    if constexpr (CPLX) {
      // periodic images (slot 0 of a dimension came from the last cell): times the conjugate phase
      // (NC = 1: the partner lane holds the other part of the same element)
      auto rot = [&](CV& u, int d, bool on) {
        CV q;
        if constexpr (NC == 2) {
          q.e[0] = P.ph.re[d] * u.e[0] + P.ph.im[d] * u.e[1];
          q.e[1] = P.ph.re[d] * u.e[1] - P.ph.im[d] * u.e[0];
        } else {
          q.e[0] = P.ph.re[d] * u.e[0] + ((li & 1) ? -P.ph.im[d] : P.ph.im[d]) * __shfl_xor(u.e[0], 1);
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) u.e[j] = on ? q.e[j] : u.e[j];
      };
      if (__any(f & kXW)) rot(a, 0, (f & kXW) != 0);
#pragma unroll
      for (int j = 0; j < NC; ++j) a.e[j] = fma(b.e[j], m2, a.e[j]);
      if ((kk & 1) == 0 && __any(f & kYW)) rot(a, 1, (f & kYW) != 0);
      if ((kk >> 1) == 0 && __any(f & kZW)) rot(a, 2, (f & kZW) != 0);
    } else {
#pragma unroll
      for (int j = 0; j < NC; ++j) a.e[j] = fma(b.e[j], m2, a.e[j]);
    }
    return a;
  };
  V4 acc[RB][NC];
  int fall = 0;    // flags of all the wave's rows
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int f = row(rb, v).flags;
      fall |= f;
      fix_odd(xr[rb][v]);
      sa[rb][v] = pair_sum(f, row(rb, v).dx, 0, sa[rb][v], sb[rb][v]);
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        asm volatile("" : "+v"(sa[rb][v].e[j]));  // formed here: frees the registers of the second slots
      }
    }
  if constexpr (PX) {
    if (tile_fptr) {
      CV xz[RB][4];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int j = 0; j < NC; ++j) xz[rb][v].e[j] = (row(rb, v).flags & kIn) ? xr[rb][v].e[j] : T(0);
      node_stash<T, NC>(xt, it, xz);
    }
  }

  // ---- the slot pairs of nodes shared in y or z, in a fixed order; a pair is visited when some lane
  // of the wave needs it, lanes that do not reload their first slot (in bounds, cached) and discard it
  auto kflags = [](int kk) { return (kk & 1 ? kY2 : 0) | (kk & 2 ? kZ2 : 0); };
  auto need = [&](int rb, int kk) {
    int anyl = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) anyl |= (row(rb, v).flags & kflags(kk)) == kflags(kk);
    return (bool)__any(anyl);
  };
  auto pair_load = [&](int kk, CV (&a)[RB][4], CV (&b)[RB][4]) {
    const int S = g.nc * g.P1;
    const int64_t kofs = (int64_t)((kk & 1 ? S : 0) + (kk & 2 ? S * S : 0)) * P.ldc;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      if (need(rb, kk)) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const NodeRow<T>& r = row(rb, v);
          const T* ya = Y + r.slot + ((r.flags & kflags(kk)) == kflags(kk) ? kofs : 0);
          a[rb][v] = load_cols<T, NC>(ya);
          b[rb][v] = load_cols<T, NC>(ya + r.dx);
        }
      }
  };
  auto pair_add = [&](int kk, const CV (&a)[RB][4], const CV (&b)[RB][4]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
      if (need(rb, kk)) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int f = row(rb, v).flags;
          const CV q = pair_sum(f, row(rb, v).dx, kk, a[rb][v], b[rb][v]);
          const T mn = (f & kflags(kk)) == kflags(kk) ? T(1) : T(0);
#pragma unroll
          for (int j = 0; j < NC; ++j) sa[rb][v].e[j] = fma(q.e[j], mn, sa[rb][v].e[j]);
        }
      }
  };

  // ---- base = m^-1/2 sum - c x (the two largest terms meet first, so that what is left of them is rounded
  // at its own size), and Ht_t Z^O over k-steps of 4 functions, KB steps of Z^O loaded ahead.  A Bloch
  // operator sums the products from zero and adds them to the base once: its k-steps, four products to an
  // element, would else each round at the size of the base (a degree-50 complex64 filter of diamond8 errs by
  // 1.02e-6 so, 1.20e-6 else); a real operator adds them onto the base.
  constexpr bool kOwn = CPLX;
  constexpr int KB = 4;
  const T* __restrict__ Zc = P.zo + colx;
  auto zload = [&](int k0, CV (&z)[KB]) {
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      z[j] = load_cols<T, NC>(Zc + (int64_t)fs[min(k0 + 4 * j + lk, FP - 1)] * ncr);
      fix_odd(z[j]);
    }
  };
  const T sz = (li & 1) ? T(1) : T(-1);  // NC = 1: sign of the partner's part
  auto hz = [&](int k0, const CV (&z)[KB]) {
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      if (k0 + 4 * j >= FP) break;
      const int f = k0 + 4 * j + lk;
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) {
        const T* h = hs + (unsigned)(((rb0 + rb) * 16 + li) * HS + f) * E;
        if constexpr (CPLX) {
          const T hr = h[0], hi = h[1];
#pragma unroll
          for (int i = 0; i < NC; ++i) acc[rb][i] = M::op(hr, z[j].e[i], acc[rb][i]);
          if constexpr (NC == 2) {
            acc[rb][0] = M::op(-hi, z[j].e[1], acc[rb][0]);
            acc[rb][1] = M::op(hi, z[j].e[0], acc[rb][1]);
          } else {
            acc[rb][0] = M::op(hi, sz * __shfl_xor(z[j].e[0], 1), acc[rb][0]);
          }
        } else {
          const T hv = h[0];
#pragma unroll
          for (int i = 0; i < NC; ++i) acc[rb][i] = M::op(hv, z[j].e[i], acc[rb][i]);
        }
      }
    }
  };
  const bool ys = __any(fall & kY2), zs = __any(fall & kZ2);
  {
    CV a[RB][4], b[RB][4];
    if (ys) {
      pair_load(1, a, b);
      pair_add(1, a, b);
    }
    if (zs) {
      pair_load(2, a, b);
      pair_add(2, a, b);
    }
    if (ys && zs) {
      pair_load(3, a, b);
      pair_add(3, a, b);
    }
  }
  CV z[KB];
  if (FP > 0) zload(0, z);
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const T msc = row(rb, v).msc;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const T base = msc * sa[rb][v].e[j] - c * xr[rb][v].e[j];
        if constexpr (kOwn) {
          sa[rb][v].e[j] = base;
          acc[rb][j][v] = T(0);
        } else {
          acc[rb][j][v] = base;
        }
      }
    }
  for (int k0 = 0; k0 < FP; k0 += 4 * KB) {
    CV zn[KB];
    if (k0 + 4 * KB < FP) zload(k0 + 4 * KB, zn);
    hz(k0, z);
#pragma unroll
    for (int j = 0; j < KB; ++j) z[j] = zn[j];
  }

  // ---- out = alpha acc - beta prev (a Bloch operator: alpha base onto that, in one rounding); rows past the
  // mesh: 0, not stored
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool ok = row(rb, v).flags & kIn;
      fix_odd(pv[rb][v]);
      CV r;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        r.e[j] = alpha * acc[rb][j][v];
        if (use_prev) r.e[j] -= beta * pv[rb][v].e[j];
        if constexpr (kOwn) r.e[j] = alpha * sa[rb][v].e[j] + r.e[j];
      }
      T* o = P.out + row(rb, v).row * P.ldo + col;
      if (ok && it.live) {
        if (NC == 2 && col + 1 < ncr)
          __builtin_memcpy(o, &r, sizeof(r));
        else if (col < ncr)
          o[0] = r.e[0];
      }
#pragma unroll
      for (int j = 0; j < NC; ++j) sa[rb][v].e[j] = ok ? r.e[j] : T(0);
    }
  if (tile_fptr && (PX || pnext)) {
    if constexpr (!PX) node_stash<T, NC>(xt, it, sa);
    node_part<T, CPLX, NC>(P, hs, HS, xt, it);
  }
}

// Node stage of real operators at one column (the auxiliary-potential conjugate gradients,
// Lanczos): one wave per coupling tile, lane = tile row, no LDS.  The slot gather takes the
// same slots in the same order as fe_node_kernel; the tile's coupling row is applied with
// one product per function in list order, and each function's partial of H^co* x is a fixed
// butterfly over the 64 rows.  Launched when every operator of the step has one column and the
// tiles couple to at most kCol1MaxFunctions functions (per-function butterflies cost more than
// the matrix-core products beyond that).
constexpr int kCol1MaxFunctions = 24;  // functions per tile up to which one column takes fe_node_col1_kernel
template <typename T>
__global__ __launch_bounds__(256) void fe_node_col1_kernel(KBatch<T> kb, int nc, int p, int n, int P1, CellCoef<T> cf,
                                                           const int32_t* __restrict__ tile_fptr,
                                                           const int32_t* __restrict__ tile_fns, int ntiles, int tm,
                                                           int pad) {
  const KP<T>& P = kb.k[blockIdx.z];
  const int tw = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // uniform per wave
  __shared__ double red[4];
  const bool live = tw < ntiles;  // a wave past the last tile repeats it and stores nothing
  const int t = live ? tw : ntiles - 1;
  const int r = (int)threadIdx.x & 63;
  int x0, y0, z0, ix, iy, iz;
  tile_origin(t, n, tm, x0, y0, z0);
  const int gv = tile_row_coords(x0, y0, z0, r, n, tm, ix, iy, iz);
  const bool ok = gv >= 0;
  const int g = ok ? gv : 0;
  T alpha, c, beta;
  step_scalars(P, alpha, c, beta);
  const T xv = ok ? P.x[(int64_t)g * P.ldx] : T(0);
  const T pv = beta != T(0) ? P.prev[(int64_t)g * P.ldo] : T(0);
  // slots of the node: (bx + {0, x2}) x (by + {0, y2}) x (bz + {0, z2}), as in fe_node_kernel
  const int qx = div_p(ix, p), rx = ix - qx * p, qy = div_p(iy, p), ry = iy - qy * p, qz = div_p(iz, p),
            rz = iz - qz * p;
  const int bx = qx * P1 + (rx ? rx + 1 : 0), by = qy * P1 + (ry ? ry + 1 : 0), bz = qz * P1 + (rz ? rz + 1 : 0);
  const bool x2 = rx == 0, y2 = ry == 0, z2 = rz == 0;
  const T msc = cf.mscale * cf.om[rx] * cf.om[ry] * cf.om[rz];
  const int S = nc * P1;
  const int64_t ldc = P.ldc, Sl = (int64_t)S * ldc, S2l = Sl * S;
  const T* __restrict__ Y0 = P.ycell + slot_index(bx, by, bz, S) * ldc;
  const T m2 = x2 ? T(1) : T(0);
  T sum = 0;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int ky = kk & 1, kz = kk >> 1;
    const bool need = ok && (ky == 0 || y2) && (kz == 0 || z2);
    const T* ya = Y0 + (need ? ky * Sl + kz * S2l : 0);
    const T* yb = x2 ? ya + ldc : ya;
    const T mn = need ? T(1) : T(0);
    sum = fma(fma(yb[0], m2, ya[0]), mn, sum);
  }
  T acc = msc * sum - c * xv;
  if (tile_fptr) {
    const int f0 = tile_fptr[t], FP = tile_fptr[t + 1] - f0;  // a multiple of 4 (padded list)
    const T* __restrict__ tv = P.tv + tile_offset(f0, t, pad) + (int64_t)r * (FP + pad);  // this row of the block
    // four functions at a time: their loads issued together, their butterflies interleaved
    for (int fb = 0; fb < FP; fb += 4) {
      T h[4], z[4], q[4];
      __builtin_memcpy(h, __builtin_assume_aligned(tv + fb, 2 * sizeof(T)), sizeof(h));  // (FP, pad and offsets are even)
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = P.zo[(int64_t)tile_fns[f0 + fb + i] * P.ncr];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc = fma(h[i], z[i], acc);
        q[i] = h[i] * xv;
      }
      // the four sums over the 64 rows: halves of the wave take two functions each, quarters one, so
      // a batch needs 7 exchanges, not 24 (the LDS permutes bound this kernel: diamond64 30.9 -> 24.9 us)
      const bool h32 = r & 32, h16 = r & 16;
      T s0 = (h32 ? q[2] : q[0]) + __shfl_xor(h32 ? q[0] : q[2], 32);
      T s1 = (h32 ? q[3] : q[1]) + __shfl_xor(h32 ? q[1] : q[3], 32);
      T sq = (h16 ? s1 : s0) + __shfl_xor(h16 ? s0 : s1, 16);
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
      if ((r & 15) == 0 && live) P.part[(int64_t)(f0 + fb + (h32 ? 2 : 0) + (h16 ? 1 : 0)) * P.ncr] = sq;
    }
  }
  T o = alpha * acc;
  if (beta != T(0)) o -= beta * pv;
  if (ok && live) P.out[(int64_t)g * P.ldo] = o;
  if (P.pq) {
    // x . out of the workgroup's rows (the conjugate gradients' p . q without a pass of its own)
    double v = ok && live ? (double)xv * (double)o : 0.0;
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) v += __shfl_xor(v, k);
    if (r == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) P.pq_part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

// First fold of the tile partials: part2[nu][ch][j] = sum of the partials of function
// nu with list positions in chunk ch (kReduceChunk entries), in list order within
// 4 interleaved groups and a fixed 4-way tree.  Chunks past the list hold 0.
constexpr int kReduceChunk = 64;

template <typename T>
__global__ __launch_bounds__(256) void enr_reduce1_kernel(KBatch<T> kb, int nch, const int32_t* __restrict__ fn_pptr,
                                                          const int32_t* __restrict__ fn_poff) {
  __shared__ T red[4][64];
  const KP<T>& P = kb.k[blockIdx.z];
  const int ncr = P.ncr;
  if ((int)blockIdx.y * 64 >= ncr) return;
  const T* __restrict__ part = P.part;
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int nu = blockIdx.x / nch, ch = blockIdx.x - nu * nch;
  const int j = blockIdx.y * 64 + lane;
  const int e1 = fn_pptr[nu + 1];
  const int es = fn_pptr[nu] + ch * kReduceChunk, ee = min(e1, es + kReduceChunk);
  // this wave's entries es + grp + 4 i, all loads issued at once; summed as two
  // interleaved chains (even i, odd i) in list order
  constexpr int EPG = kReduceChunk / 4;
  const int eg = __builtin_amdgcn_readfirstlane(es + grp);
  T v[EPG];
  if (ee > es) {
    const int jc = min(j, ncr - 1);
#pragma unroll
    for (int i = 0; i < EPG; ++i) {
      const int e = eg + 4 * i;
      const T pv = part[(int64_t)fn_poff[min(e, ee - 1)] * ncr + jc];  // clamped in-bounds entry
      // a multiply by 1 or 0 (not a select, which the compiler would turn into a branch
      // around the load) keeps all loads of the batch in flight together
      v[i] = pv * ((e < ee && j < ncr) ? T(1) : T(0));
    }
  } else {
#pragma unroll
    for (int i = 0; i < EPG; ++i) v[i] = T(0);
  }
  T s0 = 0, s1 = 0;
#pragma unroll
  for (int i = 0; i < EPG; i += 2) {
    s0 += v[i];
    s1 += v[i + 1];
  }
  red[grp][lane] = s0 + s1;
  __syncthreads();
  if (grp == 0 && j < ncr)
    P.part2[((int64_t)nu * nch + ch) * ncr + j] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// Small dense products on the enrichment rows (n = n_enr; complex interleaved when
// CPLX), 16x16 output tile per workgroup, LDS-staged K tiles.
//   mode 0: zo = S x^O       mode 1: wp = (sum of the folded tile partials) + H^oo zo
//   mode 2: out^O = alpha (S wp - c x^O) - beta prev^O
//   mode 3: zn = S out^O      (Z^O of the next recurrence step)
template <typename T, bool CPLX>
__global__ __launch_bounds__(256) void small_gemm_kernel(KBatch<T> kb, int mode, int64_t N, int n) {
  constexpr int E = CPLX ? 2 : 1;
  constexpr int TS = 16;
  __shared__ T As[TS][TS * E + 1];
  __shared__ T Bs[TS][TS * E + 1];
  const KP<T>& P = kb.k[blockIdx.z];
  const int m = P.nv;
  if ((int)blockIdx.x * TS >= m) return;
  const int k = n;
  const T* __restrict__ A = mode == 1 ? P.Hoo : P.S;
  const T* __restrict__ B = mode == 0 ? P.x + N * P.ldx
                           : mode == 3 ? P.out + N * P.ldo
                                       : (mode == 1 ? P.zo : P.wp);
  const int64_t ldb = mode == 0 ? P.ldx : mode == 3 ? P.ldo : (int64_t)P.ncr;
  const int tx = threadIdx.x % TS, ty = threadIdx.x / TS;
  const int i = blockIdx.y * TS + ty;   // row
  const int jc = blockIdx.x * TS + tx;  // column (complex element)
  T sr = 0, si = 0;
  for (int k0 = 0; k0 < k; k0 += TS) {
    for (int e = 0; e < E; ++e) {
      const int ka = k0 + tx, kr = k0 + ty;
      As[ty][tx * E + e] = (i < n && ka < k) ? A[((int64_t)i * k + ka) * E + e] : T(0);
      Bs[ty][tx * E + e] = (kr < k && jc < m) ? B[(int64_t)kr * ldb + (int64_t)jc * E + e] : T(0);
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < TS; ++kk) {
      if constexpr (!CPLX) {
        sr += As[ty][kk] * Bs[kk][tx];
      } else {
        const C2<T> t = cmul(C2<T>{As[ty][2 * kk], As[ty][2 * kk + 1]}, C2<T>{Bs[kk][2 * tx], Bs[kk][2 * tx + 1]});
        sr += t.r;
        si += t.i;
      }
    }
    __syncthreads();
  }
  if (i >= n || jc >= m) return;
  if (mode == 0 || mode == 3) {
    T* z = mode == 0 ? P.zo : P.zn;
    z[(int64_t)i * P.ncr + (int64_t)jc * E] = sr;
    if (CPLX) z[(int64_t)i * P.ncr + (int64_t)jc * E + 1] = si;
  } else if (mode == 1) {
    const T* p2 = P.part2 + (int64_t)i * P.nch * P.ncr + (int64_t)jc * E;
    T wr = 0, wi = 0;
    for (int ch = 0; ch < P.nch; ++ch) {
      wr += p2[(int64_t)ch * P.ncr];
      if (CPLX) wi += p2[(int64_t)ch * P.ncr + 1];
    }
    P.wp[(int64_t)i * P.ncr + (int64_t)jc * E] = wr + sr;
    if (CPLX) P.wp[(int64_t)i * P.ncr + (int64_t)jc * E + 1] = wi + si;
  } else {
    const int64_t ox = (N + i) * P.ldx + (int64_t)jc * E, oo = (N + i) * P.ldo + (int64_t)jc * E;
    T alpha, cst, beta;
    step_scalars(P, alpha, cst, beta);
    T r = alpha * (sr - cst * P.x[ox]);
    if (beta != T(0)) r -= beta * P.prev[oo];
    P.out[oo] = r;
    if (CPLX) {
      T r2 = alpha * (si - cst * P.x[ox + 1]);
      if (beta != T(0)) r2 -= beta * P.prev[oo + 1];
      P.out[oo + 1] = r2;
    }
  }
}

template <typename T, bool CPLX>
__global__ __launch_bounds__(1024) void enr_chain_kernel(KBatch<T> kb, ChainArgs ca) {
  extern __shared__ __align__(16) unsigned char chain_raw[];
  enr_chain<T, CPLX, kChainCols>(kb, ca, (int)blockIdx.x, chain_raw);
}

// The chain of one real column outside a recurrence: 16 lanes of a row share its sums (the chunk partials,
// or with fn_pptr the tile partials themselves, and the products), their parts added by a fixed butterfly,
// S and H^oo from memory.  enr_chain_kernel, laid out for 16 columns, computes each sum 16 times over and
// stages both matrices first: 12.3 us for 64 functions, 7.0 so.  With npq also x . out, from the node
// workgroups' partials and the enrichment rows.
// One workgroup reads both matrices, so that beyond kCol1Functions small_gemm's many workgroups are faster, and so
// is its Z^O (in the cell launch one thread takes a row of S, and no two read neighbouring entries).
// Microseconds of an application to one column, small_gemm for both -> this chain, and Z^O in the cell launch:
// auxiliary potential of 64 atoms 35 -> 25, of 125 40 -> 33, 216 51.5 -> 50.6, but 343 65 -> 86 and 512 102 ->
// 168; Kohn-Sham operators of 128 functions 48 -> 39, of 320 92 -> 108.
constexpr int kCol1Functions = 256;
template <typename T>
__global__ __launch_bounds__(1024) void enr_col1_kernel(KBatch<T> kb, int64_t N, int n,
                                                        const int32_t* __restrict__ fn_pptr,
                                                        const int32_t* __restrict__ fn_poff, int npq) {
  extern __shared__ __align__(16) unsigned char col1_raw[];
  T* Ws = reinterpret_cast<T*>(col1_raw);  // [n] W'
  __shared__ double red[16];
  const KP<T>& P = kb.k[blockIdx.z];
  const int t = (int)threadIdx.x, jl = t & 15;
  auto sum16 = [](T v) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 16);
    return v;
  };
  T alpha, cst, beta;
  step_scalars(P, alpha, cst, beta);
  double v = 0.0;
  for (int k = t; k < npq; k += 1024) v += P.pq_part[k];
  for (int i = t >> 4; i < n; i += 64) {
    T w = 0, h = 0;
    if (fn_pptr) {
      for (int e = fn_pptr[i] + jl; e < fn_pptr[i + 1]; e += 16) w += P.part[(int64_t)fn_poff[e] * P.ncr];
    } else {
#pragma unroll 4
      for (int ch = jl; ch < P.nch; ch += 16) w += P.part2[((int64_t)i * P.nch + ch) * P.ncr];
    }
#pragma unroll 4
    for (int k = jl; k < n; k += 16) h += P.Hoo[(int64_t)i * n + k] * P.zo[(int64_t)k * P.ncr];
    w = sum16(w + h);
    if (jl == 0) Ws[i] = w;
  }
  __syncthreads();
  for (int i = t >> 4; i < n; i += 64) {
    const T xv = P.x[(N + i) * P.ldx], pv = beta != T(0) ? P.prev[(N + i) * P.ldo] : T(0);
    T a = 0;
#pragma unroll 4
    for (int k = jl; k < n; k += 16) a += P.S[(int64_t)i * n + k] * Ws[k];
    a = sum16(a);
    T o = alpha * (a - cst * xv);
    if (beta != T(0)) o -= beta * pv;
    if (jl == 0) {
      P.out[(N + i) * P.ldo] = o;
      v += (double)xv * (double)o;
    }
  }
  if (!npq) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((t & 63) == 0) red[t >> 6] = v;
  __syncthreads();
  if (t == 0) {
    double sum = 0.0;
    for (int w = 0; w < 16; ++w) sum += red[w];
    *P.pq = sum;
  }
}

// diagonal test operator: out = alpha (lambda x - c x) - beta prev
template <typename T>
__global__ void diag_step_kernel(const T* __restrict__ lam, const T* __restrict__ x, const T* __restrict__ prev,
                                 T* __restrict__ out, int64_t ldx, int64_t ldo, int nv, int64_t N, T alpha, T c,
                                 T beta) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= N * nv) return;
  const int64_t g = idx / nv;
  const int vv = (int)(idx % nv);
  const int64_t o = g * ldx + vv;
  const int64_t oo = g * ldo + vv;
  T r = alpha * (lam[g] * x[o] - c * x[o]);
  if (beta != T(0)) r -= beta * prev[oo];
  out[oo] = r;
}

// ---------------------------------------------------------------------------
// Density at the quadrature points for the potential gradient:
//   dens[blk][e][q] = sum over the 64 real columns of this block of f_v psi_col(x_eq)^2,
//   psi = B (m^-1/2 theta o x)|_e + sum_nu N^O_nu(x_eq) (S x^O)_nu.
// One cell x 64 real columns per workgroup, the finite-element part in the plane layout of
// fe_cell_kernel.  The enrichment part is a product (points x functions)(functions x columns) on the
// matrix cores: with a thread per (column, points of one qx) every value N^O(x) was read from LDS for one
// product, 5 waves x 25 points x 31 functions of them per cell and the larger part of the kernel.  A wave
// takes row tiles w, w + P1, ... of 16 points and all column tiles, its accumulators start from the
// finite-element values, N^O is read once from memory, and the sum over columns needs 4 shuffles of a point's
// 16 lanes.  diamond8, 72 columns: 328 -> 163 us, of which the finite-element
// part of the second, mostly empty block of columns is about a third.  psi is float64 for float32 blocks too:
// 66 KB a workgroup for 32 (degree 4), two on a CU for five; the call with 72 float32 columns 346 -> 170 us,
// 64 columns 181 -> 98, 72 complex64 columns 1086 -> 448.
// ---------------------------------------------------------------------------
constexpr int kFnList = 128;  // enrichment functions of a cell listed at a time

template <typename T, int P1, bool CPLX>
__global__ __launch_bounds__(64 * P1) void density_kernel(
    const T* __restrict__ X, int64_t ldx, int ncr, const double* __restrict__ fw, const T* __restrict__ zo,
    CellCoef<T> cf, int nc, int p, int n, Phase3<T> ph, const int64_t* __restrict__ cph_ptr,
    const int32_t* __restrict__ cph_blk, const int64_t* __restrict__ cph_off, const int32_t* __restrict__ blk_fn0,
    const int32_t* __restrict__ blk_nf, const double* __restrict__ phi, int FMAX, int n_enr,
    double* __restrict__ dens, int64_t n_cells) {
  constexpr int NP = P1 * P1;
  constexpr int NQ = NP * P1;
  __shared__ double smem[NQ * 64];
  T(*lds)[64] = reinterpret_cast<T(*)[64]>(smem);
  __shared__ struct {
    int64_t phi;  // the function's entry of the cell's first point
    int32_t fn;   // its row of Z^O, -1: none
  } fnl[kFnList];
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int64_t e = blockIdx.x;
  const int j = min((int)blockIdx.y * 64 + lane, ncr - 1);  // columns past ncr repeat the last and are left out below
  const int cyz = (int)blockIdx.x / nc, cx = (int)blockIdx.x - cyz * nc, cz = cyz / nc, cy = cyz - cz * nc;
  // the cell's enrichment functions in a flat list, kFnList at a time; a last k-step is filled up with Z = 0
  constexpr int E = CPLX ? 2 : 1, NRT = (NQ + 15) / 16, NR = (NRT + P1 - 1) / P1, NCT = 4;
  const int64_t k0 = cph_ptr[e], k1 = cph_ptr[e + 1];
  const int nfn = (int)(k1 - k0) * FMAX, ln = lane & 15, lk = lane >> 4;
  const int jb = blockIdx.y * 64, nct = min(NCT, (ncr - jb + 15) / 16);
  auto nsteps = [&](int l0) { return (min(kFnList, nfn - l0) + 3) / 4; };
  auto list = [&](int l0) {
    for (int i = (int)threadIdx.x; i < 4 * nsteps(l0); i += 64 * P1) {
      const int l = min(l0 + i, nfn - 1), b = l / FMAX, f = l - b * FMAX;
      const int blk = cph_blk[k0 + b];
      fnl[i].phi = (cph_off[k0 + b] * NQ * FMAX + f) * E;
      fnl[i].fn = l0 + i < nfn && f < blk_nf[blk] ? blk_fn0[blk] + f : -1;
    }
  };
  // a k-step's four functions: N^O at the row tiles' points, Z of the lane's columns (a complex pair also
  // needs the swapped column: re: Re N Re z - Im N Im z, im: Re N Im z + Im N Re z)
  struct KStep {
    double pr[NR], pi[NR], z[NCT], zx[NCT];
  };
  auto load = [&](int st, KStep& k) {
    const int64_t po = fnl[4 * st + lk].phi;
    const int fn = fnl[4 * st + lk].fn;
    const T* zp = zo + (int64_t)max(fn, 0) * ncr;
#pragma unroll
    for (int c = 0; c < NCT; ++c) {
      const int jc = min(jb + 16 * c + ln, ncr - 1);
      k.z[c] = fn >= 0 ? (double)zp[jc] : 0.0;
      if (CPLX) k.zx[c] = fn >= 0 ? ((jc & 1) ? (double)zp[jc ^ 1] : -(double)zp[jc ^ 1]) : 0.0;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = min(16 * (w + r * P1) + ln, NQ - 1);
      const double* pp = phi + po + (int64_t)q * FMAX * E;
      k.pr[r] = pp[0];
      k.pi[r] = CPLX ? pp[E - 1] : 0.0;
    }
  };
  constexpr int D = CPLX ? 2 : 4;  // k-steps on their way: N^O comes from memory, and 10 waves are on a CU
  KStep ring[D];
  auto preload = [&](int l0) {
#pragma unroll
    for (int u = 0; u < D; ++u) load(min(u, nsteps(l0) - 1), ring[u]);
  };
  if (nfn > 0) list(0);
  T v[NP], t[NP];
  {
    const int az = w;
    int iz = cz * p + az;
    const bool wz = iz >= n;
    if (wz) iz -= n;
#pragma unroll
    for (int ay = 0; ay < P1; ++ay) {
      int iy = cy * p + ay;
      const bool wy = iy >= n;
      if (wy) iy -= n;
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) {
        int ix = cx * p + ax;
        const bool wx = ix >= n;
        if (wx) ix -= n;
        const int64_t g = ix + (int64_t)n * (iy + (int64_t)n * iz);
        T val;
        if constexpr (!CPLX) {
          val = X[g * ldx + j];
        } else {
          const T* px = X + g * ldx + (j & ~1);
          C2<T> z{px[0], px[1]};
          if (wx) z = cmul(z, C2<T>{ph.re[0], ph.im[0]});
          if (wy) z = cmul(z, C2<T>{ph.re[1], ph.im[1]});
          if (wz) z = cmul(z, C2<T>{ph.re[2], ph.im[2]});
          val = (j & 1) ? z.i : z.r;
        }
        v[ay * P1 + ax] = cf.mscale * cf.om[ax] * cf.om[ay] * cf.om[az] * val;
      }
    }
  }
#pragma unroll
  for (int ay = 0; ay < P1; ++ay)
#pragma unroll
    for (int qx = 0; qx < P1; ++qx) {
      T s = 0;
#pragma unroll
      for (int ax = 0; ax < P1; ++ax) s += cf.B1[qx][ax] * v[ay * P1 + ax];
      t[ay * P1 + qx] = s;
    }
#pragma unroll
  for (int qy = 0; qy < P1; ++qy)
#pragma unroll
    for (int qx = 0; qx < P1; ++qx) {
      T s = 0;
#pragma unroll
      for (int ay = 0; ay < P1; ++ay) s += cf.B1[qy][ay] * t[ay * P1 + qx];
      lds[(w * P1 + qy) * P1 + qx][lane] = s;
    }
  __syncthreads();
  if (nfn > 0) preload(0);
#pragma unroll
  for (int az = 0; az < P1; ++az)
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) t[az * P1 + qy] = lds[(az * P1 + qy) * P1 + w][lane];
  // psi of the finite-element part at the points, float64, in the transpose's place
  __syncthreads();
  double(*psi)[64] = reinterpret_cast<double(*)[64]>(smem);
#pragma unroll
  for (int qz = 0; qz < P1; ++qz)
#pragma unroll
    for (int qy = 0; qy < P1; ++qy) {
      T s = 0;
#pragma unroll
      for (int az = 0; az < P1; ++az) s += cf.B1[qz][az] * t[az * P1 + qy];
      psi[(qz * P1 + qy) * P1 + w][lane] = (double)s;
    }
  double fv[NCT];
#pragma unroll
  for (int c = 0; c < NCT; ++c) {
    const int jc = jb + 16 * c + ln;
    fv[c] = jc < ncr ? fw[CPLX ? jc >> 1 : jc] : 0.0;
  }
  typedef Mfma<double>::V4 V4;
  V4 acc[NR][NCT];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < NCT; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int q = 16 * (w + r * P1) + Mfma<double>::row(lane, v);
        acc[r][c][v] = q < NQ ? psi[q][16 * c + ln] : 0.0;
      }
  for (int l0 = 0; l0 < nfn; l0 += kFnList) {
    if (l0) {
      __syncthreads();
      list(l0);
      __syncthreads();
      preload(l0);
    }
    const int steps = nsteps(l0);
    for (int st = 0; st < steps; st += D)
#pragma unroll
      for (int u = 0; u < D; ++u) {
        if (st + u >= steps) break;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          if (w + r * P1 >= NRT) break;
#pragma unroll
          for (int c = 0; c < NCT; ++c) {
            if (c >= nct) break;
            acc[r][c] = Mfma<double>::op(ring[u].pr[r], ring[u].z[c], acc[r][c]);
            if (CPLX) acc[r][c] = Mfma<double>::op(ring[u].pi[r], ring[u].zx[c], acc[r][c]);
          }
        }
        load(min(st + u + D, steps - 1), ring[u]);
      }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (w + r * P1 >= NRT) break;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double sum = 0.0;
#pragma unroll
      for (int c = 0; c < NCT; ++c)
        if (jb + 16 * c + ln < ncr) sum += fv[c] * acc[r][c][v] * acc[r][c][v];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 16);
      const int q = 16 * (w + r * P1) + Mfma<double>::row(lane, v);
      if (ln == 0 && q < NQ) dens[((int64_t)blockIdx.y * n_cells + e) * NQ + q] = sum;
    }
  }
}

struct GW {
  double w[8];
};
// mode 0: out = W s (the potential gradient); 1: out = s (the density); 2: out += s
__global__ void density_final_kernel2(const double* __restrict__ dens, int nblk, int64_t total, int P1, GW gw,
                                      double h3, double* __restrict__ out, int mode) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= total) return;
  const int nq = P1 * P1 * P1;
  const int q = (int)(t % nq);
  double s = 0;
  for (int b = 0; b < nblk; ++b) s += dens[(int64_t)b * total + t];
  if (mode == 0) {
    const double W = h3 * gw.w[q % P1] * gw.w[(q / P1) % P1] * gw.w[q / (P1 * P1)];
    out[t] = W * s;
  } else if (mode == 1) {
    out[t] = s;
  } else {
    out[t] += s;
  }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <typename T>
const CellCoef<T>& coef(const oefe_op_s* op);
template <>
const CellCoef<double>& coef<double>(const oefe_op_s* op) { return op->cd; }
template <>
const CellCoef<float>& coef<float>(const oefe_op_s* op) { return op->cf; }

template <typename T>
struct DevPtrs {
  const T *WV, *S, *Hoo, *lambda, *tv;
};
template <typename T>
DevPtrs<T> devptrs(const oefe_op_s* op);
template <>
DevPtrs<double> devptrs<double>(const oefe_op_s* op) {
  return {op->d.WV, op->d.S, op->d.Hoo, op->d.lambda, op->d.tile_val};
}
template <>
DevPtrs<float> devptrs<float>(const oefe_op_s* op) {
  return {op->d.WVf, op->d.Sf, op->d.Hoof, op->d.lambdaf, op->d.tile_valf};
}

template <typename T, int P1, int CW, bool CPLX>
void launch_cell_cw(const oefe_op_s* op, const KBatch<T>& kb, int max_ncr, hipStream_t s) {
  constexpr int CPT = 64 / CW;
  dim3 grid((unsigned)cdiv(op->n_cells, CPT), (unsigned)cdiv(max_ncr, CW), (unsigned)kb.nk);
  hipLaunchKernelGGL((fe_cell_kernel<T, P1, CW, CPLX>), grid, dim3(64 * P1), 0, s, kb, coef<T>(op), op->nc, op->p,
                     op->n, op->n_cells);
}

template <typename T, int P1, bool CPLX>
void launch_cell_p(const oefe_op_s* op, const KBatch<T>& kb, int max_ncr, int cw, hipStream_t s) {
  switch (cw) {
    case 64: launch_cell_cw<T, P1, 64, CPLX>(op, kb, max_ncr, s); break;
    case 32: launch_cell_cw<T, P1, 32, CPLX>(op, kb, max_ncr, s); break;
    case 16: launch_cell_cw<T, P1, 16, CPLX>(op, kb, max_ncr, s); break;
    default: launch_cell_cw<T, P1, 8, CPLX>(op, kb, max_ncr, s); break;
  }
}

template <typename T, int P1, bool CPLX>
void launch_cell_lanes(const oefe_op_s* op, const KBatch<T>& kb, int max_ncr, hipStream_t s, const ChainArgs& ca) {
  constexpr int CWc = lanes_cw<P1>();
  const int nch = (int)cdiv(max_ncr, CWc);
  dim3 grid((unsigned)(cdiv(op->n_cells, 4) * nch + ca.nblk), 1, (unsigned)kb.nk);
  const bool chain = ca.nblk && !ca.zo_only;
  auto go = [&](auto uf) {
    constexpr bool UF = decltype(uf)::value;
    using F = CellFirst;
    const bool own = ca.nblk ? cell_lanes_own_lds<T, P1, UF>(F::zo) : cell_lanes_own_lds<T, P1, UF>(F::none);
    const size_t tile = own ? 0 : cell_lanes_lds_bytes<T, P1>();  // dynamic LDS
    const size_t lds =
        chain ? std::max(cell_lanes_lds_bytes<T, P1>(), enr_chain_lds_bytes<T, CPLX>(ca.n, kChainColsCell)) : tile;
    auto* kernel = chain     ? &fe_cell_lanes_kernel<T, P1, CPLX, UF, F::chain>
                   : ca.nblk ? &fe_cell_lanes_kernel<T, P1, CPLX, UF, F::zo>
                             : &fe_cell_lanes_kernel<T, P1, CPLX, UF, F::none>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), lds, s, kb, coef<T>(op), op->nc, op->p, op->n, op->n_cells, nch, ca);
  };
  if constexpr (CPLX) {
    if (op->uform) {  // the operators of a batch share the form (checked by the batched entry points)
      go(std::true_type{});
      return;
    }
  }
  go(std::false_type{});
}

// The planes-in-lanes kernel forms row offsets within a z-plane of X and of the node-slot
// grid in 32 bits from 24-bit products: n^2 ldx and S^2 ldc below 2^31 (S = nc (p+1)).
template <typename T>
bool lanes_offsets_fit(const oefe_op_s* op, const KBatch<T>& kb) {
  const int64_t S = (int64_t)op->nc * op->P1, n = op->n;
  for (int q = 0; q < kb.nk; ++q) {
    const int64_t ldx = kb.k[q].ldx, ldc = kb.k[q].ldc;
    if (ldx * n * n >= (int64_t(1) << 31) || ldc * S * S >= (int64_t(1) << 31)) return false;
  }
  return true;
}

// Whether a recurrence's step runs its enrichment chain as the first blocks of the cell launch, in
// stream order, instead of on the side stream beside the cell and node stages: two launches a step (three
// with the fold of many partials) against three or four and four event calls.  Microseconds a step, side
// stream -> in the cell launch: one atom, 4 k elements 32.3 -> 18.8, 0.8 M 34.4 -> 27.8; eight atoms
// 0.34 M 36.9 -> 30.2 (float32 42.5 -> 25.1), 1.6 M 47.1 -> 42.9, 4.1 M 87.0 -> 82.1, 8.0 M 169.2 -> 168.0
// (float32 98.7 -> 96.6); four k-points of 17 M elements each 1703 -> 1726 and 1880 -> 1953
// (periodic-function form): there the fold, not the waits, is what the side stream hides.
// Every cell workgroup of such a launch holds the chain's LDS and registers (complex128 degree 2: 124 for 64).
// One complex128 k-point of eight atoms, 16 / 24 / 32 functions (three workgroups a CU or more): degree 2,
// 1.0 M elements 52 -> 47 and 3.1 M 92 -> 91; degree 4, 5.3 M 124 -> 117 and 8.2 M 226 -> 222.  With 40
// functions (59 KB of LDS: two workgroups a CU): degree 2, 0.44 M 48 -> 38, 1.0 M 59 -> 60, 1.8 M 66 -> 70;
// degree 3, 0.66 M 47 -> 41, 1.0 M 54 -> 55, 1.8 M 60 -> 67; degree 4, 1.1 M 55 -> 52, 1.6 M 72 -> 72.5, 2.0 M
// 70 -> 61, 2.8 M 84 -> 81, 3.5 M 115 -> 117, 5.3 M 145 -> 142, 8.2 M 261 -> 265.
// Complex64 (29 KB): never slower up to 8 M.
template <typename T, bool CPLX>
bool chain_in_cell(const oefe_op_s* op, const KBatch<T>& kb, bool bf16) {
  if (bf16 || op->n_enr < 1 || (op->tune_cw != 0 && !op->uform) || !lanes_offsets_fit(op, kb)) return false;
  const size_t lds = enr_chain_lds_bytes<T, CPLX>(op->n_enr, kChainColsCell);
  if (lds > 64 * 1024) return false;
  int64_t elems = 0;
  for (int q = 0; q < kb.nk; ++q) {
    if (kb.k[q].nv < 2) return false;  // one column folds its partials in another order
    elems += op->N * kb.k[q].ncr;
  }
  // (two workgroups a CU instead of seven and four of degree 2 and 3; degree 4 has three)
  return elems <= (op->P1 == 5 || 3 * lds <= 160 * 1024 ? kChainInCellElems : (int64_t)3 << 18);
}

// cw = 0: planes-in-lanes kernel; 8, 16, 32, 64: plane-per-wave kernel with cw columns per cell
template <typename T, int P1>
void launch_cell_cells(const oefe_op_s* op, const KBatch<T>& kb, hipStream_t s, const ChainArgs& ca) {
  constexpr int CWc = lanes_cw<P1>();
  hipLaunchKernelGGL((fe_cell_cells_kernel<T, P1>), dim3((unsigned)(cdiv(op->n_cells, 4 * CWc) + ca.nblk), 1, (unsigned)kb.nk),
                     dim3(256), 0, s, kb, coef<T>(op), op->nc, op->p, op->n, op->n_cells, ca);
}

template <typename T, bool CPLX>
void launch_cell(const oefe_op_s* op, const KBatch<T>& kb, int max_ncr, int cw, hipStream_t s, const ChainArgs& ca) {
  if constexpr (!CPLX) {
    if (max_ncr == 1) {  // one real column: cells in the lanes, whatever the tuned shape
      switch (op->P1) {
        case 3: launch_cell_cells<T, 3>(op, kb, s, ca); break;
        case 4: launch_cell_cells<T, 4>(op, kb, s, ca); break;
        default: launch_cell_cells<T, 5>(op, kb, s, ca); break;
      }
      return;
    }
  }
  if (op->uform) {
    // only the planes-in-lanes kernel carries the periodic-function form's first-derivative
    // term; oefe_op_create_uform checks that its 32-bit offsets fit the mesh
    cw = 0;
  } else if (cw == 0 && !lanes_offsets_fit(op, kb)) {
    cw = 16;
  }
  if (cw == 0) {
    switch (op->P1) {
      case 3: launch_cell_lanes<T, 3, CPLX>(op, kb, max_ncr, s, ca); break;
      case 4: launch_cell_lanes<T, 4, CPLX>(op, kb, max_ncr, s, ca); break;
      default: launch_cell_lanes<T, 5, CPLX>(op, kb, max_ncr, s, ca); break;
    }
    return;
  }
  switch (op->P1) {
    case 3: launch_cell_p<T, 3, CPLX>(op, kb, max_ncr, cw, s); break;
    case 4: launch_cell_p<T, 4, CPLX>(op, kb, max_ncr, cw, s); break;
    default: launch_cell_p<T, 5, CPLX>(op, kb, max_ncr, cw, s); break;
  }
}

// part kernel, or node kernel with part of this step's X (px) or of its result (pnext)
enum class NodeRun { part, node_px, node, node_pnext };
template <typename T, bool CPLX, int NC>
int launch_node_nc(const oefe_op_s* op, const KBatch<T>& kb, int max_ncr, NodeRun run, hipStream_t s) {
  NodeMesh g{op->nc, op->p, op->n, op->P1, (int)op->N, op->tile_mode, tile_count(op->n, op->tile_mode),
             op->n_enr > 0 ? op->tile_fpmax : 0, op->tile_pad, 1, 1};
  // Column groups per workgroup (W, two waves each; the tuner's, else 1, 2 or 4), and whether items run
  // across tile ends (the blocks of up to ntl tiles in LDS) or tiles are padded to whole workgroups: the
  // shape with the most waves resident on a CU (16 by their registers, and the LDS), less the padding's
  // idle ones.  At equal counts 4 groups share a block in float64 (diamond64, 320 columns: 2930 us
  // against 3560 with 2) and 2 in float32 (1430 against 1480); else the wider of equals.  Small launches take
  // narrower workgroups than that, 2 groups below five workgroups of 4 to four CUs (complex128, whose blocks are
  // the largest: one to a CU) and 1 where that still is less than a group to a CU: a CU then copies fewer blocks before
  // its work can start.  Applications in microseconds with 1, 2 and 4 groups: float64, 216 tiles of 1 group
  // (8 vectors) 32, 33, 35; 92 x 3 30, 29, 33; 216 x 3 37, 38, 39; 216 x 5 48, 43, 47; 343 x 5 57, 56, 53.  Complex128,
  // 92 x 3 42, 40, 44; 216 x 3 58, 49, 51; 216 x 5 71, 64, 60.  Complex64, 216 x 1 36.5, 37, 42; 216 x 2 42, 41, 45.
  const int G = (int)cdiv(max_ncr, 16 * NC);
  const int fixed = op->tune_cb > 0 ? std::max(1, std::min(kNodeGroups, op->tune_cb / 16)) : 0;
  int64_t items = 0;  // (tile, column group) pairs of the launch
  for (int q = 0; q < kb.nk; ++q) items += g.ntiles * cdiv(kb.k[q].ncr, 16 * NC);
  int W = 1;
  double best = 0;
  for (int w : {1, 2, 4}) {
    if (fixed ? w != (fixed == 3 ? 2 : fixed) : w > 1 && items < (w == 2 ? 256 : CPLX && sizeof(T) == 8 ? 1024 : 1280)) continue;
    int ntl = 1;
    for (int q = 0; q < kb.nk; ++q) ntl = std::max(ntl, node_tiles((int)cdiv(kb.k[q].ncr, 16 * NC), w));
    for (int span = 0; span < 2; ++span) {
      const size_t l = node_lds<T, CPLX, NC>(g.fpmax, g.pad, span ? ntl : 1, w).total;
      if (l > 160 * 1024) continue;
      const double eff = span ? 1.0 : (double)G / (double)(cdiv(G, w) * w);
      const double score = eff * 2 * w * std::min<int64_t>(8 / w, 160 * 1024 / (int64_t)l) +
                           (w == (sizeof(T) == 8 ? 4 : 2) ? 1e-3 : 1e-4 * w);
      if (score > best) {
        best = score;
        W = w;
        g.span = span;
        g.ntl = span ? ntl : 1;
      }
    }
  }
  const size_t lds = node_lds<T, CPLX, NC>(g.fpmax, g.pad, g.ntl, W).total;
  int64_t nwg = 1;
  for (int q = 0; q < kb.nk; ++q) {
    const int64_t gq = cdiv(kb.k[q].ncr, 16 * NC);
    nwg = std::max(nwg, cdiv(g.ntiles * (g.span ? gq : cdiv(gq, W) * W), W));
  }
  const int32_t* fptr = op->n_enr > 0 ? op->d.tile_fptr : nullptr;
  const dim3 grid((unsigned)nwg, 1u, (unsigned)kb.nk), block(128 * W);
  if (run == NodeRun::part) {
    if (allow_dynamic_lds(reinterpret_cast<const void*>(&fe_part_kernel<T, CPLX, NC>), lds) != hipSuccess)
      return OEFE_EDEVICE;
    hipLaunchKernelGGL((fe_part_kernel<T, CPLX, NC>), grid, block, lds, s, kb, g, fptr, op->d.tile_fns);
    return OEFE_OK;
  }
  auto go = [&](auto kernel) {
    if (allow_dynamic_lds(reinterpret_cast<const void*>(kernel), lds) != hipSuccess) return (int)OEFE_EDEVICE;
    hipLaunchKernelGGL(kernel, grid, block, lds, s, kb, g, coef<T>(op), fptr, op->d.tile_fns,
                       run == NodeRun::node_pnext ? 1 : 0);
    return (int)OEFE_OK;
  };
  if (run == NodeRun::node_px) return go(&fe_node_kernel<T, CPLX, NC, true>);
  return go(&fe_node_kernel<T, CPLX, NC, false>);
}

// float32: two columns per lane, so that a wave's row segments fill 128-byte lines; a single real
// column takes one per lane, and so do real blocks that groups of 32 columns would pad by more than 15 %
// over groups of 16 (diamond8, 72 columns: 62 -> 59 us and a degree 96.5 -> 93.5; a column's sums are the same)
template <typename T, bool CPLX>
int launch_node(const oefe_op_s* op, const KBatch<T>& kb, int max_ncr, NodeRun run, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    int min_ncr = max_ncr;
    for (int q = 0; q < kb.nk; ++q) min_ncr = std::min(min_ncr, kb.k[q].ncr);
    const bool narrow = !CPLX && 20 * cdiv(max_ncr, 32) * 32 > 23 * cdiv(max_ncr, 16) * 16;
    if (CPLX || (min_ncr >= 2 && !narrow)) return launch_node_nc<T, CPLX, 2>(op, kb, max_ncr, run, s);
  }
  if constexpr (sizeof(T) == 8 || !CPLX) return launch_node_nc<T, CPLX, 1>(op, kb, max_ncr, run, s);
  return OEFE_EINVAL;
}

inline int reduce_chunks(const oefe_op_s* op) { return std::max(1, (int)cdiv(op->fn_smax, kReduceChunk)); }

// Steps of several operators sharing one mesh and enrichment layout, in lockstep.
void launch_cell_bf16(const oefe_op_s* op, const KBatch<float>& kb, hipStream_t s) {
  const size_t lds = 3 * (size_t)kBf16MatElems * sizeof(uint16_t) + 128 * (3 * sizeof(int) + sizeof(float));
  if (allow_dynamic_lds(reinterpret_cast<const void*>(&fe_cell_bf16_kernel), lds) != hipSuccess) return;
  int cus = 256;
  int dev = 0;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  hipLaunchKernelGGL(fe_cell_bf16_kernel, dim3((unsigned)std::max(1, cus / kb.nk), 1, (unsigned)kb.nk), dim3(768),
                     lds, s, kb, op->d.bf_mats, op->cf, op->nc, op->p, op->n, op->P1, op->n_cells);
}

}  // namespace

// Whether a step of one real column outside a recurrence can form x . out as it goes: the flat node
// kernel and the chain in one launch.
bool pq_in_step(const oefe_op_s* op) {
  return !op->cplx && !op->diagonal && op->n_enr > 0 && op->tile_fpmax <= kCol1MaxFunctions &&
         op->n_enr <= kCol1Functions;
}
int64_t pq_partials(const oefe_op_s* op) { return cdiv(tile_count(op->n, op->tile_mode), 4); }

namespace {

template <typename T, bool CPLX>
int apply_step_batch_impl(const oefe_op_s* const* ops, const KBatch<T>& kb, hipStream_t s, const Overlap* ov,
                          bool bf16) {
  const oefe_op_s* op = ops[0];
  int max_ncr = 0, max_nv = 0;
  for (int q = 0; q < kb.nk; ++q) {
    max_ncr = std::max(max_ncr, kb.k[q].ncr);
    max_nv = std::max(max_nv, kb.k[q].nv);
    if (ops[q]->uform != op->uform) return OEFE_EINVAL;  // one form per batch
  }
  // the periodic-function form runs on the planes-in-lanes cell kernel only
  if (op->uform && !lanes_offsets_fit(op, kb)) return OEFE_EUNSUPPORTED;
  const unsigned nk = (unsigned)kb.nk;
  const int nO = op->n_enr;
  const bool ovl = ov != nullptr && nO > 0;
  // optional HIP events around one stage (oefe_kernel_timer), on the stream it runs on
  auto timed = [&](int kind, hipStream_t st, auto&& launch) {
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const bool on = op->timer_kind == kind && hipEventCreate(&ev0) == hipSuccess && hipEventCreate(&ev1) == hipSuccess;
    if (on) (void)hipEventRecord(ev0, st);
    launch();
    if (on) {
      (void)hipEventRecord(ev1, st);
      op->timer_events.emplace_back(ev0, ev1);
    }
  };
  ChainArgs ca{};
  auto cell_stage = [&] {
    timed(OEFE_TIMER_CELL, s, [&] {
      if constexpr (std::is_same<T, float>::value && !CPLX) {
        if (bf16) {
          launch_cell_bf16(op, kb, s);
          return;
        }
      }
      launch_cell<T, CPLX>(op, kb, max_ncr, op->tune_cw, s, ca);
    });
  };
  const dim3 gg((unsigned)cdiv(max_nv, 16), (unsigned)cdiv(nO, 16), nk);
  const size_t clds = enr_chain_lds_bytes<T, CPLX>(nO);
  const bool one_chain =
      nO > 0 && clds <= 96 * 1024 &&
      allow_dynamic_lds(reinterpret_cast<const void*>(&enr_chain_kernel<T, CPLX>), clds) == hipSuccess;
  // few partials per function (small meshes): the chain folds them itself, one launch fewer
  const bool direct = (one_chain || (!CPLX && !ovl && max_nv == 1 && nO <= kCol1Functions)) && op->fn_smax <= kReduceChunk;
  const bool pq = kb.k[0].pq != nullptr;
  const bool col1_chain = !CPLX && !ovl && max_nv == 1 && nO > 0 && nO <= kCol1Functions;
  if (pq && !(col1_chain && pq_in_step(op))) return OEFE_EINVAL;
  // fold of the tile partials, and the chain that forms W' from it and writes the enrichment rows of
  // out (and, in an overlapped recurrence, Z^O of the next step), on stream se
  auto fold = [&](hipStream_t se) {
    if (direct) return;
    const int nch = reduce_chunks(op);
    hipLaunchKernelGGL((enr_reduce1_kernel<T>), dim3((unsigned)(nO * nch), (unsigned)cdiv(max_ncr, 64), nk),
                       dim3(256), 0, se, kb, nch, op->d.fn_pptr, op->d.fn_poff);
  };
  auto chain = [&](hipStream_t se) {
    if (col1_chain) {
      if constexpr (!CPLX)
        hipLaunchKernelGGL((enr_col1_kernel<T>), dim3(1, 1, nk), dim3(1024), (size_t)nO * sizeof(T), se, kb, op->N, nO,
                           direct ? op->d.fn_pptr : nullptr, op->d.fn_poff, pq ? (int)pq_partials(op) : 0);
    } else if (one_chain) {
      const ChainArgs c{op->N, nO, (ovl && !ov->last) ? 1 : 0, direct ? op->d.fn_pptr : nullptr, op->d.fn_poff, 0, false};
      hipLaunchKernelGGL((enr_chain_kernel<T, CPLX>), dim3((unsigned)cdiv(max_nv, kChainCols), 1, nk), dim3(1024), clds,
                         se, kb, c);
    } else {
      hipLaunchKernelGGL((small_gemm_kernel<T, CPLX>), gg, dim3(256), 0, se, kb, 1, op->N, nO);
      hipLaunchKernelGGL((small_gemm_kernel<T, CPLX>), gg, dim3(256), 0, se, kb, 2, op->N, nO);
      if (ovl && !ov->last) hipLaunchKernelGGL((small_gemm_kernel<T, CPLX>), gg, dim3(256), 0, se, kb, 3, op->N, nO);
    }
  };
  // one column: the flat kernel where tiles couple to few functions (the auxiliary-potential
  // operator, one function per atom: 23 % less time per conjugate-gradient iteration on
  // diamond64); the Kohn-Sham operator's ~50 functions per tile stay on the matrix cores
  const bool col1 = !CPLX && !ovl && max_ncr == 1 && op->tile_fpmax <= kCol1MaxFunctions;
  // A recurrence forms each step's partials Ht_t^* X with the X that the previous step wrote, while it
  // is in registers; its first step, from X itself, before the node stage.
  const bool ahead = ovl, inl = ahead && one_chain && chain_in_cell<T, CPLX>(op, kb, bf16);
  int rc = OEFE_OK;
  // outside a recurrence Z^O is formed by the first blocks of the cell launch (of the two kernels that
  // take them): one launch fewer, 25.1 -> 22.8 us for the application to one atom's 8 vectors
  const bool zo_in_cell = nO > 0 && !ovl && !bf16 && (max_nv > 1 || nO <= kCol1Functions) &&
                          ((!CPLX && max_ncr == 1) || op->uform || (op->tune_cw == 0 && lanes_offsets_fit(op, kb)));
  if (zo_in_cell) {
    const int nblk = (int)cdiv((int64_t)nO * max_nv, 256);
    ca = ChainArgs{op->N, nO, 0, nullptr, nullptr, max_ncr == 1 ? nblk : (int)cdiv(nblk, 8) * 8, true};
  }
  if (nO > 0 && (!ovl || ov->first) && !zo_in_cell) {
    hipLaunchKernelGGL((small_gemm_kernel<T, CPLX>), gg, dim3(256), 0, s, kb, 0, op->N, nO);
    if (ahead) {
      rc = launch_node<T, CPLX>(op, kb, max_ncr, NodeRun::part, s);
      if (rc) return rc;
      fold(s);
      if (!inl) {
        (void)hipEventRecord(ov->ev_node, s);
        (void)hipStreamWaitEvent(ov->side, ov->ev_node, 0);
      }
    }
  }
  if (inl)
    ca = ChainArgs{op->N, nO, ov->last ? 0 : 1, direct ? op->d.fn_pptr : nullptr, op->d.fn_poff,
                   (int)cdiv(cdiv(max_nv, kChainColsCell), 8) * 8, false};  // (whole rounds of the XCDs)
  // The chain of this step (folded partials, Z^O and enrichment rows are there) beside its cell and
  // node stages: the next step's Z^O goes to a buffer of its own
  if (nO > 0 && ahead && !inl) {
    chain(ov->side);
    if (direct) (void)hipEventRecord(ov->ev_zo, ov->side);  // the partials are read
  }
  cell_stage();
  // this step's Z^O is there and its partials are folded
  if (ovl && nO > 0 && !inl && (direct || !ov->first)) (void)hipStreamWaitEvent(s, ov->ev_zo, 0);
  if (col1) {
    if constexpr (!CPLX) {
      const int ntiles = tile_count(op->n, op->tile_mode);
      timed(OEFE_TIMER_NODE, s, [&] {
        hipLaunchKernelGGL((fe_node_col1_kernel<T>), dim3((unsigned)cdiv(ntiles, 4), 1u, (unsigned)kb.nk), dim3(256), 0, s,
                           kb, op->nc, op->p, op->n, op->P1, coef<T>(op), op->n_enr > 0 ? op->d.tile_fptr : nullptr,
                           op->d.tile_fns, ntiles, op->tile_mode, op->tile_pad);
      });
    }
  } else {
    // (a Bloch operator's node kernel is also its coupling stage)
    const int kind = CPLX && nO > 0 && op->timer_kind == OEFE_TIMER_COUPLING ? OEFE_TIMER_COUPLING : OEFE_TIMER_NODE;
    const NodeRun run = !ahead ? NodeRun::node_px : ov->last ? NodeRun::node : NodeRun::node_pnext;
    timed(kind, s, [&] { rc = launch_node<T, CPLX>(op, kb, max_ncr, run, s); });
    if (rc) {  // the chain is queued: the caller's stream waits for ev_zo
      if (nO > 0 && ahead && !inl) (void)hipEventRecord(ov->ev_zo, ov->side);
      return rc;
    }
  }
  if (inl) {
    if (!ov->last) fold(s);
  } else if (nO > 0 && ahead) {
    // the fold of the next step's partials beside its cell stage
    if (!ov->last) {
      (void)hipEventRecord(ov->ev_node, s);
      (void)hipStreamWaitEvent(ov->side, ov->ev_node, 0);
      fold(ov->side);
    }
    if (!direct) {
      (void)hipEventRecord(ov->ev_zo, ov->side);
      if (ov->last) (void)hipStreamWaitEvent(s, ov->ev_zo, 0);
    }
  } else if (nO > 0) {
    fold(s);
    chain(s);
  }
  return hipGetLastError() == hipSuccess ? OEFE_OK : OEFE_EDEVICE;
}

template <typename T>
KP<T> make_kp(const oefe_op_s* op, const T* x, int64_t ld, const T* prev, T* out, int64_t ldout, int nv,
              double alpha, double c, double beta, const StepWork& w) {
  const bool cx = op->cplx;
  const DevPtrs<T> dp = devptrs<T>(op);
  KP<T> P{};
  P.x = x;
  P.prev = prev;
  P.out = out;
  P.ldx = cx ? 2 * ld : ld;
  P.ldo = cx ? 2 * ldout : ldout;
  P.nv = nv;
  P.ncr = cx ? 2 * nv : nv;
  P.ycell = (T*)w.ycell;
  P.ldc = w.ldc;
  P.zo = (T*)w.zo;
  P.zn = (T*)w.zn;
  P.part = (T*)w.part;
  P.part2 = (T*)w.part2;
  P.nch = reduce_chunks(op);
  P.wp = (T*)w.wp;
  P.pq = w.pq;
  P.pq_part = w.pq_part;
  P.wv = dp.WV;
  P.tv = dp.tv;
  P.S = dp.S;
  P.Hoo = dp.Hoo;
  P.alpha = (T)alpha;
  P.c = (T)c;
  P.beta = (T)beta;
  P.sc = nullptr;
  for (int d = 0; d < 3; ++d) {
    P.ph.re[d] = (T)op->phase[d][0];
    P.ph.im[d] = (T)op->phase[d][1];
    P.uk[d] = (T)op->uk[d];
  }
  return P;
}

template <typename T, int P1, bool CPLX>
void launch_density(const oefe_op_s* op, const T* x, int64_t ldx, int ncr, const double* f, const T* zo, double* dens,
                    hipStream_t s) {
  Phase3<T> ph;
  for (int d = 0; d < 3; ++d) {
    ph.re[d] = (T)op->phase[d][0];
    ph.im[d] = (T)op->phase[d][1];
  }
  dim3 grid((unsigned)op->n_cells, (unsigned)cdiv(ncr, 64));
  hipLaunchKernelGGL((density_kernel<T, P1, CPLX>), grid, dim3(64 * P1), 0, s, x, ldx, ncr, f, zo, coef<T>(op),
                     op->nc, op->p, op->n, ph, op->d.cph_ptr, op->d.cph_blk, op->d.cph_off, op->d.blk_fn0,
                     op->d.blk_nf, op->d.phi, op->FMAX, op->n_enr, dens, op->n_cells);
}

}  // namespace

// Node-slot grid elements: n_cells nd rows of ldc, then a padding of one row plus 32 elements.  The
// node kernel reads the columns of a row without clamping them to ncr: at most ncr + 30 for a group
// of up to 32 columns that starts below ncr, so the reads past the last row's end stay inside the padding
// (ncr <= ldc).
static size_t slot_grid_elems(const oefe_op_s* op, int ldc) {
  return (size_t)op->n_cells * op->nd * ldc + (size_t)ldc + 32;
}

size_t step_work_bytes(const oefe_op_s* op, int elem_bytes, bool cplx, int nv, int* ldc_out) {
  const int ncr = cplx ? 2 * nv : nv;
  // rows of the node-slot grid: a multiple of 8 columns, except one real column, whose slots
  // are then contiguous (every cell kernel stores only columns below ncr; the node kernels'
  // reads past the column stay inside the grid's padding)
  const int ldc = ncr == 1 ? 1 : (int)cdiv(ncr, 8) * 8;
  if (ldc_out) *ldc_out = ldc;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  size_t bytes = 0;
  if (!op->diagonal) bytes += al(slot_grid_elems(op, ldc) * elem_bytes);
  bytes += 2 * al((size_t)std::max(op->n_enr, 1) * ncr * elem_bytes);             // zo, zn
  bytes += al((size_t)std::max<int64_t>(op->tile_slots, 1) * ncr * elem_bytes);  // part
  bytes += al((size_t)std::max(op->n_enr, 1) * reduce_chunks(op) * ncr * elem_bytes);  // part2
  bytes += al((size_t)std::max(op->n_enr, 1) * ncr * elem_bytes);                 // wp
  return bytes;
}

StepWork carve_step_work(const oefe_op_s* op, int elem_bytes, bool cplx, int nv, void* work) {
  StepWork w{};
  const int ncr = cplx ? 2 * nv : nv;
  int ldc;
  step_work_bytes(op, elem_bytes, cplx, nv, &ldc);
  w.ldc = ldc;
  auto al = [](size_t b) { return (b + 255) / 256 * 256; };
  char* p = (char*)work;
  if (!op->diagonal) {
    w.ycell = p;
    p += al(slot_grid_elems(op, ldc) * elem_bytes);
  }
  w.zo = p;
  p += al((size_t)std::max(op->n_enr, 1) * ncr * elem_bytes);
  w.zn = p;
  p += al((size_t)std::max(op->n_enr, 1) * ncr * elem_bytes);
  w.part = p;
  p += al((size_t)std::max<int64_t>(op->tile_slots, 1) * ncr * elem_bytes);
  w.part2 = p;
  p += al((size_t)std::max(op->n_enr, 1) * reduce_chunks(op) * ncr * elem_bytes);
  w.wp = p;
  return w;
}

template <typename T>
int apply_step(const oefe_op_s* op, bool bf16, const T* x, int64_t ld, const T* prev, T* out, int64_t ldo, int nv,
               double alpha, double c, double beta, const StepWork& w, hipStream_t s, const Overlap* ov,
               const double* sc) {
  // BF16 cell stage: real operators with float32 vectors and the dense-cell matrices
  if (bf16 && (sizeof(T) != 4 || op->cplx || op->diagonal || !op->d.bf_mats)) return OEFE_EUNSUPPORTED;
  if (!x || !out || (beta != 0.0 && !prev)) return OEFE_EINVAL;  // prev is read only when beta != 0
  if (sc && op->diagonal) return OEFE_EUNSUPPORTED;
  if (op->diagonal) {
    const DevPtrs<T> dp = devptrs<T>(op);
    const int64_t tot = op->N * nv;
    hipLaunchKernelGGL((diag_step_kernel<T>), dim3((unsigned)cdiv(tot, 256)), dim3(256), 0, s, dp.lambda, x, prev,
                       out, ld, ldo, nv, op->N, (T)alpha, (T)c, (T)beta);
    return hipGetLastError() == hipSuccess ? OEFE_OK : OEFE_EDEVICE;
  }
  KBatch<T> kb{};
  kb.nk = 1;
  kb.k[0] = make_kp<T>(op, x, ld, prev, out, ldo, nv, alpha, c, beta, w);
  kb.k[0].sc = sc;
  const oefe_op_s* ops[1] = {op};
  if (op->cplx) return apply_step_batch_impl<T, true>(ops, kb, s, ov, false);
  return apply_step_batch_impl<T, false>(ops, kb, s, ov, bf16);
}

template int apply_step<double>(const oefe_op_s*, bool, const double*, int64_t, const double*, double*, int64_t, int,
                                double, double, double, const StepWork&, hipStream_t, const Overlap*, const double*);
template int apply_step<float>(const oefe_op_s*, bool, const float*, int64_t, const float*, float*, int64_t, int,
                               double, double, double, const StepWork&, hipStream_t, const Overlap*, const double*);

// The scalars of an m-step filter from device bounds (a, b, a0), in the order and arithmetic
// of the host recurrence: step 0 (s1 / e, c, 0), step k (2 s_k+1 / e, c, s_k s_k+1) with
// e = (b - a) / 2, c = (b + a) / 2, s1 = e / (a0 - c), s_k+1 = 1 / (2 / s1 - s_k).  Bounds
// that violate a0 < a < b give zero scalars and status {OEFE_EINVAL, 0}; else {0, -1}.
__global__ void cheb_scalars_kernel(const double* __restrict__ bounds, int m, double* __restrict__ out,
                                    int32_t* __restrict__ status) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const double a = bounds[0], b = bounds[1], a0 = bounds[2];
  const bool ok = a < b && a0 < a && isfinite(a) && isfinite(b) && isfinite(a0);
  const double e = (b - a) / 2.0, c = (b + a) / 2.0;
  const double s1 = e / (a0 - c);
  out[0] = ok ? s1 / e : 0.0;
  out[1] = ok ? c : 0.0;
  out[2] = 0.0;
  double sig = s1;
  for (int k = 1; k < m; ++k) {
    const double sn = 1.0 / (2.0 / s1 - sig);
    out[3 * k] = ok ? 2.0 * sn / e : 0.0;
    out[3 * k + 1] = ok ? c : 0.0;
    out[3 * k + 2] = ok ? sig * sn : 0.0;
    sig = sn;
  }
  if (status) {
    status[0] = ok ? 0 : OEFE_EINVAL;
    status[1] = ok ? -1 : 0;
  }
}

int cheb_scalars(const double* bounds, int m, double* out, int32_t* status, hipStream_t s) {
  hipLaunchKernelGGL(cheb_scalars_kernel, dim3(1), dim3(64), 0, s, bounds, m, out, status);
  return hipGetLastError() == hipSuccess ? OEFE_OK : OEFE_EDEVICE;
}

template <typename T>
int apply_step_batch(const oefe_op_s* const* ops, int nk, bool bf16, const T* const* x, const int64_t* ld,
                     const T* const* prev, T* const* out, const int64_t* ldo, const int* nv, const double* alpha,
                     const double* c, const double* beta, const StepWork* w, hipStream_t s, const Overlap* ov) {
  if (bf16)
    for (int q = 0; q < nk; ++q)
      if (sizeof(T) != 4 || ops[q]->cplx || ops[q]->diagonal || !ops[q]->d.bf_mats) return OEFE_EUNSUPPORTED;
  for (int q = 0; q < nk; ++q)  // the kernels read prev only when beta is nonzero
    if (!x[q] || !out[q] || (beta[q] != 0.0 && !prev[q])) return OEFE_EINVAL;
  for (int q0 = 0; q0 < nk; q0 += KMAX) {
    KBatch<T> kb{};
    kb.nk = std::min(KMAX, nk - q0);
    for (int q = 0; q < kb.nk; ++q)
      kb.k[q] = make_kp<T>(ops[q0 + q], x[q0 + q], ld[q0 + q], prev[q0 + q], out[q0 + q], ldo[q0 + q], nv[q0 + q],
                           alpha[q0 + q], c[q0 + q], beta[q0 + q], w[q0 + q]);
    // overlap only when the whole batch is one launch group
    const Overlap* o = nk <= KMAX ? ov : nullptr;
    const int rc = ops[0]->cplx ? apply_step_batch_impl<T, true>(ops + q0, kb, s, o, false)
                                : apply_step_batch_impl<T, false>(ops + q0, kb, s, o, bf16);
    if (rc) return rc;
  }
  return OEFE_OK;
}

template int apply_step_batch<double>(const oefe_op_s* const*, int, bool, const double* const*, const int64_t*,
                                      const double* const*, double* const*, const int64_t*, const int*, const double*,
                                      const double*, const double*, const StepWork*, hipStream_t, const Overlap*);
template int apply_step_batch<float>(const oefe_op_s* const*, int, bool, const float* const*, const int64_t*,
                                     const float* const*, float* const*, const int64_t*, const int*, const double*,
                                     const double*, const double*, const StepWork*, hipStream_t, const Overlap*);

template <typename T>
int zo_only(const oefe_op_s* op, const T* x, int64_t ld, int nv, T* zo, int ncr, hipStream_t s) {
  if (op->n_enr == 0) return OEFE_OK;
  StepWork w{};
  w.zo = zo;
  KBatch<T> kb{};
  kb.nk = 1;
  kb.k[0] = make_kp<T>(op, x, ld, nullptr, nullptr, ld, nv, 0, 0, 0, w);
  kb.k[0].ncr = ncr;
  if (op->cplx)
    hipLaunchKernelGGL((small_gemm_kernel<T, true>), dim3((unsigned)cdiv(nv, 16), (unsigned)cdiv(op->n_enr, 16), 1),
                       dim3(256), 0, s, kb, 0, op->N, op->n_enr);
  else
    hipLaunchKernelGGL((small_gemm_kernel<T, false>), dim3((unsigned)cdiv(nv, 16), (unsigned)cdiv(op->n_enr, 16), 1),
                       dim3(256), 0, s, kb, 0, op->N, op->n_enr);
  return hipGetLastError() == hipSuccess ? OEFE_OK : OEFE_EDEVICE;
}

template int zo_only<double>(const oefe_op_s*, const double*, int64_t, int, double*, int, hipStream_t);
template int zo_only<float>(const oefe_op_s*, const float*, int64_t, int, float*, int, hipStream_t);

template <typename T>
int density_partial(const oefe_op_s* op, const T* x, int64_t ld, int nv, const double* f, const T* zo, int ncr,
                    double* dens, hipStream_t s) {
  const bool c = op->cplx;
  const int64_t ldx = c ? 2 * ld : ld;
  switch (op->P1) {
    case 3: c ? launch_density<T, 3, true>(op, x, ldx, ncr, f, zo, dens, s) : launch_density<T, 3, false>(op, x, ldx, ncr, f, zo, dens, s); break;
    case 4: c ? launch_density<T, 4, true>(op, x, ldx, ncr, f, zo, dens, s) : launch_density<T, 4, false>(op, x, ldx, ncr, f, zo, dens, s); break;
    default: c ? launch_density<T, 5, true>(op, x, ldx, ncr, f, zo, dens, s) : launch_density<T, 5, false>(op, x, ldx, ncr, f, zo, dens, s); break;
  }
  return hipGetLastError() == hipSuccess ? OEFE_OK : OEFE_EDEVICE;
}

int density_final(const oefe_op_s* op, const double* dens, int nblk, double* dEdV, hipStream_t s, int mode) {
  const int64_t total = op->n_cells * op->nq;
  GW gw;
  for (int i = 0; i < 8; ++i) gw.w[i] = i < op->P1 ? op->gauss_w[i] : 0.0;
  const double h3 = (op->h / 2) * (op->h / 2) * (op->h / 2);
  hipLaunchKernelGGL(density_final_kernel2, dim3((unsigned)cdiv(total, 256)), dim3(256), 0, s, dens, nblk, total,
                     op->P1, gw, h3, dEdV, mode);
  return hipGetLastError() == hipSuccess ? OEFE_OK : OEFE_EDEVICE;
}

template int density_partial<double>(const oefe_op_s*, const double*, int64_t, int, const double*, const double*, int,
                                     double*, hipStream_t);
template int density_partial<float>(const oefe_op_s*, const float*, int64_t, int, const double*, const float*, int,
                                    double*, hipStream_t);

}  // namespace oefe
