// Solver helpers on the sparse covariance (Section 2.5): SpMV / SpMM,
// dot products, the low-rank preconditioner, the posterior variance and
// Taylor log-det drivers, and stochastic Lanczos quadrature of ln det A
// from the CG coefficients, for gfx950.  The block CG itself is in cg.hip.
//
// Caller-facing SpMM on row-major [n][R] blocks: R == 1 takes the SpMV
// kernel (16 lanes per row), even R the 32-column slab kernel of cg.hip,
// odd R a one-wavefront-per-row kernel whose 64 lanes hold 64 consecutive
// columns.  Reductions are deterministic (fixed-order block partials).
#include <algorithm>
#include <cmath>
#include <vector>

#include "kernel_math.hpp"
#include "sdgp_internal.hpp"

namespace sdgp {

namespace {

// y = sum_k val[k] X[col[k], rc] over one CSR row (the calling wave's row).
// The row's entries are loaded 64 at a time by the lanes and broadcast with
// readlane; 16 gathers are issued before their products are summed so that
// enough loads are in flight to cover the cache latency.
__device__ __forceinline__ double row_dot(const int64_t k0, const int64_t k1, const int32_t* __restrict__ col,
                                          const double* __restrict__ val, const double* __restrict__ Xc,
                                          const int64_t R) {
  const int lane = lane_id();
  double acc = 0.0;
  for (int64_t kb = k0; kb < k1; kb += kWave) {
    const int64_t k = kb + lane;
    int cj = 0;
    double vj = 0.0;
    if (k < k1) { cj = col[k]; vj = val[k]; }
    const int cnt = (int)min((int64_t)kWave, k1 - kb);
    int j = 0;
    for (; j + 16 <= cnt; j += 16) {
      double xv[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) xv[u] = Xc[(int64_t)readlane_i32(cj, j + u) * R];
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += readlane_f64(vj, j + u) * xv[u];
    }
    for (; j + 4 <= cnt; j += 4) {
      double xv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) xv[u] = Xc[(int64_t)readlane_i32(cj, j + u) * R];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc += readlane_f64(vj, j + u) * xv[u];
    }
    for (; j < cnt; ++j) acc += readlane_f64(vj, j) * Xc[(int64_t)readlane_i32(cj, j) * R];
  }
  return acc;
}

// Rows handled by the calling wave under an XCD-aware mapping: the grid's
// blocks are dealt round-robin to the 8 XCDs, so XCD x (blocks with
// blockIdx.x % 8 == x) takes the x-th eighth of the rows and all its waves
// sweep that range together, keeping the gathered neighbour rows in the
// XCD's own L2.  gridDim.x must be a multiple of 8.
struct RowSweep {
  int64_t a, hi, step;
  __device__ RowSweep(int64_t n, int waves_per_block) {
    const int xcd = blockIdx.x & 7;
    const int64_t bi = blockIdx.x >> 3;
    const int64_t nbx = gridDim.x >> 3;
    const int64_t nx = (n + 7) >> 3;
    const int64_t lo = xcd * nx;
    hi = min(n, lo + nx);
    step = nbx * waves_per_block;
    a = lo + bi * waves_per_block + (threadIdx.x >> 6);
  }
};

// Plain SpMM of columns that do not make whole 16-byte pairs, 35 and more of them or
// few rows: Y = A X (one wave per row, lanes over a 64-column chunk).
__global__ __launch_bounds__(256) void k_spmm(int64_t n, const int64_t* __restrict__ row_ptr,
                                              const int32_t* __restrict__ col, const double* __restrict__ val,
                                              const double* __restrict__ X, int R, double* __restrict__ Y) {
  const int rc = blockIdx.y * kWave + lane_id();
  const int rcc = rc < R ? rc : R - 1;
  for (RowSweep w(n, 4); w.a < w.hi; w.a += w.step) {
    const int64_t a = w.a;
    const double v = row_dot(row_ptr[a], row_ptr[a + 1], col, val, X + rcc, R);
    if (rc < R) Y[a * (int64_t)R + rc] = v;
  }
}

// SpMV (one right-hand side): 32 lanes per row, 8 rows per 256-thread block;
// each lane loads 4 of its row's (column, value) pairs (stride 32) and then
// issues their 4 gathers together.  Rows are dealt XCD-aware as in RowSweep;
// many small blocks (about four row groups each) keep the tail short.
constexpr int kSpmvLanes = 32;
constexpr int kSpmvU = 4;
__global__ __launch_bounds__(256) void k_spmv(int64_t n, const int64_t* __restrict__ row_ptr,
                                              const int32_t* __restrict__ col, const double* __restrict__ val,
                                              const double* __restrict__ x, double* __restrict__ y) {
  constexpr int G = 256 / kSpmvLanes;
  const int sub = threadIdx.x & (kSpmvLanes - 1);
  const int r = threadIdx.x / kSpmvLanes;
  const int xcd = blockIdx.x & 7;
  const int64_t bi = blockIdx.x >> 3, nbx = gridDim.x >> 3;
  const int64_t nx = (n + 7) >> 3, lo = xcd * nx, hi = min(n, lo + nx);
  for (int64_t base = lo + bi * G; base < hi; base += nbx * G) {
    const int64_t a = base + r;
    double acc = 0.0;
    if (a < hi) {
      const int64_t k1 = row_ptr[a + 1];
      for (int64_t k0 = row_ptr[a] + sub; k0 < k1; k0 += kSpmvLanes * kSpmvU) {
        int cj[kSpmvU];
        double vj[kSpmvU];
#pragma unroll
        for (int u = 0; u < kSpmvU; ++u) {
          const int64_t k = k0 + kSpmvLanes * u;
          cj[u] = k < k1 ? col[k] : 0;
          vj[u] = k < k1 ? val[k] : 0.0;
        }
        double xv[kSpmvU];
#pragma unroll
        for (int u = 0; u < kSpmvU; ++u) xv[u] = x[cj[u]];
#pragma unroll
        for (int u = 0; u < kSpmvU; ++u) acc += vj[u] * xv[u];
      }
    }
#pragma unroll
    for (int o = kSpmvLanes / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kSpmvLanes);
    if (a < hi && sub == 0) y[a] = acc;
  }
}

// SpMV with paired loads: 32 lanes per row, two rows per wavefront, 8 rows
// per 256-thread block (measured at 1M points, ~90 entries per row: 32
// lanes 0.341 ms, 16 lanes 0.366, 8 lanes 0.479, 64 lanes 0.383; two rows
// per lane group or more pairs in flight no faster).  A row's entries are
// read in 16-byte-aligned pairs
// (one 8-byte column pair and one 16-byte value pair per lane; pair halves
// outside the row are masked), two pairs per lane in flight and their four
// gathers issued together.  A pair is only loaded whole when its second
// entry exists in the arrays (nnz = row_ptr[n]); the last entry of the
// matrix is read alone.  Needs val 16-byte and col 8-byte aligned.
constexpr int kSpw = 32;
__global__ __launch_bounds__(256) void k_spmv_w(int64_t n, const int64_t* __restrict__ row_ptr,
                                                const int32_t* __restrict__ col, const double* __restrict__ val,
                                                const double* __restrict__ x, double* __restrict__ y) {
  constexpr int G = 256 / kSpw;
  const int64_t nnz = row_ptr[n];
  const int sub = threadIdx.x & (kSpw - 1);
  const int r = threadIdx.x / kSpw;
  const int xcd = blockIdx.x & 7;
  const int64_t bi = blockIdx.x >> 3, nbx = gridDim.x >> 3;
  const int64_t nx = (n + 7) >> 3, lo = xcd * nx, hi = min(n, lo + nx);
  for (int64_t base = lo + bi * G; base < hi; base += nbx * G) {
    const int64_t a = base + r;
    double acc = 0.0;
    if (a < hi) {
      const int64_t k0 = row_ptr[a], k1 = row_ptr[a + 1];
      for (int64_t e = (k0 & ~(int64_t)1) + 2 * sub; e < k1; e += 4 * kSpw) {
        int cj[4] = {0, 0, 0, 0};
        double vj[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int64_t ep = e + 2 * kSpw * h;
          if (ep < k1) {
            if (ep + 1 < nnz) {
              const int2 cc = *reinterpret_cast<const int2*>(col + ep);
              const double2 vv = *reinterpret_cast<const double2*>(val + ep);
              cj[2 * h] = cc.x;
              cj[2 * h + 1] = cc.y;
              vj[2 * h] = ep >= k0 ? vv.x : 0.0;
              vj[2 * h + 1] = ep + 1 < k1 ? vv.y : 0.0;
            } else {
              cj[2 * h] = col[ep];
              vj[2 * h] = ep >= k0 ? val[ep] : 0.0;
            }
          }
        }
        double xv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) xv[u] = x[cj[u]];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += vj[u] * xv[u];
      }
    }
#pragma unroll
    for (int o = kSpw / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kSpw);
    if (a < hi && sub == 0) y[a] = acc;
  }
}

// ------------------------------------------------------------ utilities
__global__ void k_dot_part(const double* __restrict__ a, int64_t sa, const double* __restrict__ b,
                           int64_t sb, int64_t n, double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    s += a[i * sa] * b[i * sb];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void k_probe_bits(const int32_t* __restrict__ perm, int64_t n, int P, uint64_t seed,
                             uint64_t* __restrict__ bits) {
  const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (s >= n) return;
  uint64_t m = 0;
  for (int p = 0; p < P; ++p) {
    const uint64_t k = ((uint64_t)p << 32) + (uint64_t)perm[s] + 1ull;
    if (splitmix64_at(seed, k) >> 63) m |= 1ull << p;
  }
  bits[s] = m;
}

// Column 0 of the row-major block B [n][ld].
__global__ void k_put_column(const double* __restrict__ v, int64_t n, int ld, double* __restrict__ B) {
  const int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (a < n) B[a * ld] = v[a];
}

// mean[t] = sum_b kappa[t, b] X[b][0], one wavefront per test row.
__global__ void k_mean_rows(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                            const double* __restrict__ val, int64_t nq, int ld, const double* __restrict__ X,
                            double* __restrict__ mean) {
  const int64_t t = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (t >= nq) return;
  double s = 0.0;
  for (int64_t k = rp[t] + lane_id(); k < rp[t + 1]; k += kWave) s += val[k] * X[(int64_t)col[k] * ld];
  s = wave_sum(s);
  if (lane_id() == 0) mean[t] = s;
}

// Dense right-hand sides B[b][j] = kappa[t0 + j, b] for a chunk of Rc test rows
// (B, row stride ld, zeroed beforehand; every (b, j) is written at most once).
__global__ void k_scatter_chunk(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                const double* __restrict__ val, int64_t t0, int Rc, int64_t nq, int ld,
                                double* __restrict__ B) {
  const int64_t j = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (j >= Rc || t0 + j >= nq) return;
  const int64_t t = t0 + j;
  for (int64_t k = rp[t] + lane_id(); k < rp[t + 1]; k += kWave) B[(int64_t)col[k] * ld + j] = val[k];
}

// var[t] = kxx[t] - sum_b kappa[t, b] V[b][j] for the chunk's test rows.
__global__ void k_rowdot_chunk(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                               const double* __restrict__ val, int64_t t0, int Rc, int64_t nq, int ld,
                               const double* __restrict__ V, const double* __restrict__ kxx,
                               double* __restrict__ var) {
  const int64_t j = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) >> 6;
  if (j >= Rc || t0 + j >= nq) return;
  const int64_t t = t0 + j;
  double s = 0.0;
  for (int64_t k = rp[t] + lane_id(); k < rp[t + 1]; k += kWave) s += val[k] * V[(int64_t)col[k] * ld + j];
  s = wave_sum(s);
  if (lane_id() == 0) var[t] = kxx[t] - s;
}

// Gershgorin bound: per-block partial maxima of sum_b |A_ab| over rows.
__global__ void k_rowabs_max(const int64_t* __restrict__ rp, const double* __restrict__ val, int64_t n,
                             double* __restrict__ part) {
  __shared__ double sh[256];
  double m = 0.0;
  for (int64_t a = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; a < n; a += (int64_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int64_t k = rp[a]; k < rp[a + 1]; ++k) s += fabs(val[k]);
    m = fmax(m, s);
  }
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + o]);
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Rademacher probe block Z[n][P] (caller row perm[a]) and V = Z.
__global__ void k_taylor_init(const int32_t* __restrict__ perm, int64_t n, int P, uint64_t seed,
                              double* __restrict__ Z, double* __restrict__ V) {
  const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (idx >= n * P) return;
  const int64_t a = idx / P;
  const int p = (int)(idx % P);
  const uint64_t k = ((uint64_t)p << 32) + (uint64_t)perm[a] + 1ull;
  const double z = (splitmix64_at(seed, k) >> 63) ? -1.0 : 1.0;
  Z[idx] = z;
  V[idx] = z;
}

// V <- V - W / alpha (= C V) and partial sums of Z . V.
__global__ void k_taylor_step(int64_t len, const double* __restrict__ Z, const double* __restrict__ W,
                              double* __restrict__ V, double inv_alpha, double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < len; i += (int64_t)gridDim.x * blockDim.x) {
    const double v = V[i] - W[i] * inv_alpha;
    V[i] = v;
    s += Z[i] * v;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

}  // namespace

void posterior_solve(Ctx* c, const Csr& A, const Sorted& s, const double* ys, const Csr& K0, const double* kxx,
                     double rtol, int max_iter, const Precond* pc, double* mean, double* var, bool* converged) {
  const int64_t n = A.n, n0 = K0.n;
  const char* bad = "CG met p^T A p <= 0: the covariance is not positive definite";
  *converged = true;
  // Column CG: y is column 0 of the first chunk, and a chunk fills the GPU's
  // CUs with columns (chunks of 64 leave most of them idle).  Its right-hand
  // sides, solutions and working copies of them (three blocks of 1024 columns at
  // most) are taken only from memory that is free twice over; otherwise the
  // narrow chunks, which need a sixteenth.
  const int wide = (int)std::min<int64_t>(1023, n0);
  const int n1 = pc ? pc->n1 : 0;
  bool cols = column_cg_chosen(c) && column_cg_applies(c, n, A.nnz, 1 + wide, n1, false, max_iter);
  if (cols) {
    const size_t block = sizeof(double) * (size_t)(n + 63) * (1 + wide);
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) == hipSuccess)
      cols = c->growth(S_POST, block) + c->growth(S_CG_P, block) + c->growth(S_CG_X, block) <= 0.5 * (double)free_b;
  }
  const int step = cols ? wide : kWave;
  if (!cols) {
    CgResult cg = block_cg(c, A, s, ys, PK_NONE, 0, 0, rtol, max_iter, nullptr, 0, pc, false, nullptr);
    if (cg.not_spd) throw Error(SDGP_ERR_NOT_SPD, bad);
    *converged = cg.converged;
    spmm(c, K0, cg.X, 1, mean);
  }
  for (int64_t t0 = 0; t0 < n0; t0 += step) {
    const int Rt = (int)std::min<int64_t>(step, n0 - t0);
    const int y0 = cols && t0 == 0 ? 1 : 0;        // columns before the test columns
    const int Rc = Rt + y0;
    double* B = c->get<double>(S_POST, (size_t)n * Rc);
    SDGP_HIP(hipMemsetAsync(B, 0, (size_t)n * Rc * sizeof(double), c->stream));
    if (y0) {
      k_put_column<<<(unsigned)((n + 255) / 256), 256, 0, c->stream>>>(ys, n, Rc, B);
      SDGP_CHECK_LAUNCH();
    }
    const unsigned g = (unsigned)((Rt + 3) / 4);
    k_scatter_chunk<<<g, 256, 0, c->stream>>>(K0.row_ptr, K0.col, K0.val, t0, Rt, n0, Rc, B + y0);
    SDGP_CHECK_LAUNCH();
    // (every chunk by the solver that was chosen, the last and narrower one too)
    CgResult cg = cols ? column_cg(c, {CgMember{A, pc}}, s, nullptr, PK_DENSE, Rc, 0, rtol, rtol, max_iter, B, false)[0]
                       : block_cg(c, A, s, nullptr, PK_DENSE, 0, 0, rtol, max_iter, B, Rc, pc, false, nullptr);
    if (cg.not_spd) throw Error(SDGP_ERR_NOT_SPD, bad);
    if (!cg.converged) *converged = false;
    if (y0) {
      k_mean_rows<<<(unsigned)((n0 + 3) / 4), 256, 0, c->stream>>>(K0.row_ptr, K0.col, K0.val, n0, Rc, cg.X, mean);
      SDGP_CHECK_LAUNCH();
    }
    k_rowdot_chunk<<<g, 256, 0, c->stream>>>(K0.row_ptr, K0.col, K0.val, t0, Rt, n0, Rc, cg.X + y0, kxx, var);
    SDGP_CHECK_LAUNCH();
  }
}

double logdet_taylor(Ctx* c, const Csr& A, const Sorted& s, int P, int terms, uint64_t seed, double* alpha_out) {
  require(P >= 1 && P <= 4096, "probes must be 1..4096");
  require(terms >= 1, "terms must be >= 1");
  const int64_t n = A.n;
  const int nbm = (int)std::min<int64_t>(1024, (n + 255) / 256);
  double* pm = c->get<double>(S_RED_PART, std::max(nbm, 1024));
  k_rowabs_max<<<nbm, 256, 0, c->stream>>>(A.row_ptr, A.val, n, pm);
  SDGP_CHECK_LAUNCH();
  std::vector<double> hm(nbm);
  SDGP_HIP(hipMemcpyAsync(hm.data(), pm, nbm * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  double alpha = 0.0;
  for (double v : hm) alpha = std::max(alpha, v);
  require(alpha > 0.0 && std::isfinite(alpha), "matrix has no positive row sums");
  *alpha_out = alpha;
  double acc = 0.0;
  if (taylor_terms(c, A, s, P, terms, seed, alpha, &acc)) return (double)n * std::log(alpha) - acc;
  const size_t len = (size_t)n * P;
  double* Z = c->get<double>(S_CG_X, len);
  double* V = c->get<double>(S_CG_R, len);
  double* W = c->get<double>(S_CG_Q, len);
  k_taylor_init<<<(unsigned)((len + 255) / 256), 256, 0, c->stream>>>(s.perm, n, P, seed, Z, V);
  SDGP_CHECK_LAUNCH();
  const int nb = (int)std::min<int64_t>(1024, ((int64_t)len + 255) / 256);
  std::vector<double> hp((size_t)nb * terms);
  double* part = c->get<double>(S_RED_OUT, (size_t)nb * terms);
  for (int k = 1; k <= terms; ++k) {
    spmm(c, A, V, P, W);
    k_taylor_step<<<nb, 256, 0, c->stream>>>((int64_t)len, Z, W, V, 1.0 / alpha, part + (size_t)(k - 1) * nb);
    SDGP_CHECK_LAUNCH();
  }
  SDGP_HIP(hipMemcpyAsync(hp.data(), part, hp.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  for (int k = 1; k <= terms; ++k) {
    double t = 0.0;
    for (int b = 0; b < nb; ++b) t += hp[(size_t)(k - 1) * nb + b];
    acc += t / P / k;
  }
  return (double)n * std::log(alpha) - acc;
}

void spmm(Ctx* c, const Csr& A, const double* X, int R, double* Y) {
  require(R >= 1 && R <= (1 << 20), "R must be in 1..2^20");
  const int64_t cu = std::max(8, c->cu_count);
  if (R == 1) {
    const bool aligned = (reinterpret_cast<uintptr_t>(A.val) % 16) == 0 && (reinterpret_cast<uintptr_t>(A.col) % 8) == 0;
    if (aligned) {
      // 8 rows per block step, up to 65528 blocks
      int64_t blocks = std::min<int64_t>((A.n + 7) / 8, 65528);
      blocks = std::max<int64_t>(8, (blocks + 7) / 8 * 8);
      k_spmv_w<<<(unsigned)blocks, 256, 0, c->stream>>>(A.n, A.row_ptr, A.col, A.val, X, Y);
      SDGP_CHECK_LAUNCH();
      return;
    }
    // 8 rows per block step, up to 32768 blocks
    int64_t blocks = std::min<int64_t>((A.n + 7) / 8, 32768);
    blocks = std::max<int64_t>(8, (blocks + 7) / 8 * 8);
    k_spmv<<<(unsigned)blocks, 256, 0, c->stream>>>(A.n, A.row_ptr, A.col, A.val, X, Y);
    SDGP_CHECK_LAUNCH();
    return;
  }
  // Slabs of 32 columns for whole 16-byte pairs, and for other operands of one
  // slab (33 columns: 0.49 -> 0.24 ms at 200,000 rows in sorted order; in random
  // order 3 / 17 / 25 / 33 columns 0.44 / 0.47 / 0.56 / 0.66 -> 0.26 / 0.43 / 0.55
  // / 0.67).  Two slabs of unaligned pairs lose to k_spmm's one chunk of 64 in
  // random order, where the gathers come from HBM (49 columns 1.23 against 0.87).
  // Few rows leave the GPU idle with four of them to a wavefront, and a long row is
  // a chain four times as long as with a wavefront to itself: 31 columns, rows of
  // 1000 entries, slabs against k_spmm 74 / 36 us at 1000 rows, 74 / 63 at 2000, 92
  // / 119 at 4000 (256 entries: 21 / 11, 21 / 18, 21 / 32); so up to 12 rows a CU.
  const bool pairs = R % 2 == 0 && (reinterpret_cast<uintptr_t>(X) % 16) == 0 && (reinterpret_cast<uintptr_t>(Y) % 16) == 0;
  if (pairs || (R <= 33 && A.n > 12 * cu && A.n <= 0x7fffffffLL)) {
    spmm_slab(c, A, X, R, Y, pairs);
    return;
  }
  const int chunks = (R + kWave - 1) / kWave;
  int64_t blocks = std::min<int64_t>((A.n + 3) / 4, std::max<int64_t>(8, cu * 8 / chunks));
  blocks = std::max<int64_t>(8, (blocks + 7) / 8 * 8);
  dim3 grid((unsigned)blocks, (unsigned)chunks);
  k_spmm<<<grid, 256, 0, c->stream>>>(A.n, A.row_ptr, A.col, A.val, X, R, Y);
  SDGP_CHECK_LAUNCH();
}

double dot_device(Ctx* c, const double* a, int64_t sa, const double* b, int64_t sb, int64_t n) {
  const int nb = (int)std::min<int64_t>(256, (n + 255) / 256);
  double* part = c->get<double>(S_RED_PART, nb);
  k_dot_part<<<nb, 256, 0, c->stream>>>(a, sa, b, sb, n, part);
  SDGP_CHECK_LAUNCH();
  std::vector<double> hp(nb);
  SDGP_HIP(hipMemcpyAsync(hp.data(), part, nb * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  double s = 0.0;
  for (int i = 0; i < nb; ++i) s += hp[i];
  return s;
}

void probe_bits(Ctx* c, const Sorted& s, int P, uint64_t seed, uint64_t* zbits) {
  k_probe_bits<<<(unsigned)((s.n + 255) / 256), 256, 0, c->stream>>>(s.perm, s.n, P, seed, zbits);
  SDGP_CHECK_LAUNCH();
}

namespace {

// Gram matrix F^T F: block b accumulates rows [b*slab, (b+1)*slab) staged
// 64 at a time in LDS; thread t owns the pairs idx = t, t+256, ...
__global__ __launch_bounds__(256) void k_gram(const double* __restrict__ F, int64_t n, int n1, int64_t slab,
                                              double* __restrict__ part) {
  // population form: member blockIdx.z's F (stride n * n1) and partials
  F += (int64_t)blockIdx.z * n * n1;
  part += (int64_t)blockIdx.z * gridDim.x * n1 * n1;
  __shared__ double rows[64 * kMaxN1];
  const int np = n1 * n1;
  double acc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0.0;
  const int64_t lo = blockIdx.x * slab, hi = min(n, lo + slab);
  for (int64_t a0 = lo; a0 < hi; a0 += 64) {
    const int cnt = (int)min((int64_t)64, hi - a0);
    __syncthreads();
    for (int idx = threadIdx.x; idx < cnt * n1; idx += blockDim.x) rows[idx] = F[a0 * n1 + idx];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int idx = threadIdx.x + q * 256;
      if (idx < np) {
        const int i = idx / n1, j = idx % n1;
        double s = 0.0;
        for (int k = 0; k < cnt; ++k) s += rows[k * n1 + i] * rows[k * n1 + j];
        acc[q] += s;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int idx = threadIdx.x + q * 256;
    if (idx < np) part[(int64_t)blockIdx.x * np + idx] = acc[q];
  }
}

}  // namespace

namespace {

// c and ln det M of the low-rank preconditioner, without the bump part.
Precond lowrank_base(const KParams& kp, int64_t n, const double* F) {
  Precond pc;
  const double psi0 = kp.core == SDGP_CORE_KSTAT ? 0.26596152026762178529 : 1.0;
  pc.c = kp.sigma2 * psi0 + kp.noise;
  require(pc.c > 0.0, "the low-rank preconditioner needs sigma2 psi(0) + noise_var > 0");
  pc.n1 = kp.n1;
  pc.F = F;
  if (kp.n1 == 0) pc.logdetM = (double)n * std::log(pc.c);
  return pc;
}

// From the Gram partials hp[nbk][n1*n1]: S = c I + F^T F, its Cholesky
// factor, ln det M and S^{-1} (into Si, host).
void lowrank_finish(Precond& pc, int64_t n, int64_t nbk, const double* hp, std::vector<double>& Si) {
  const int n1 = pc.n1;
  const int np = n1 * n1;
  std::vector<double> S((size_t)np, 0.0), L((size_t)np, 0.0);
  Si.assign((size_t)np, 0.0);
  for (int64_t bb = 0; bb < nbk; ++bb)
    for (int q = 0; q < np; ++q) S[q] += hp[bb * np + q];
  for (int i = 0; i < n1; ++i) S[i * n1 + i] += pc.c;
  double logdetS = 0.0;
  for (int j = 0; j < n1; ++j) {
    double d = S[j * n1 + j];
    for (int k = 0; k < j; ++k) d -= L[j * n1 + k] * L[j * n1 + k];
    require(d > 0.0, "preconditioner factor is not positive definite");
    const double ljj = std::sqrt(d);
    L[j * n1 + j] = ljj;
    logdetS += 2.0 * std::log(ljj);
    for (int i = j + 1; i < n1; ++i) {
      double v = S[i * n1 + j];
      for (int k = 0; k < j; ++k) v -= L[i * n1 + k] * L[j * n1 + k];
      L[i * n1 + j] = v / ljj;
    }
  }
  for (int col = 0; col < n1; ++col) {  // solve L L^T x = e_col
    std::vector<double> y(n1, 0.0);
    for (int i = 0; i < n1; ++i) {
      double v = (i == col) ? 1.0 : 0.0;
      for (int k = 0; k < i; ++k) v -= L[i * n1 + k] * y[k];
      y[i] = v / L[i * n1 + i];
    }
    for (int i = n1 - 1; i >= 0; --i) {
      double v = y[i];
      for (int k = i + 1; k < n1; ++k) v -= L[k * n1 + i] * Si[k * n1 + col];
      Si[i * n1 + col] = v / L[i * n1 + i];
    }
  }
  pc.logdetM = (double)(n - n1) * std::log(pc.c) + logdetS;
}

}  // namespace

Precond lowrank_precond(Ctx* c, const Sorted& s, const KParams& kp, const Bumps& b) {
  const int64_t n = s.n;
  Precond pc = lowrank_base(kp, n, b.F);
  const int n1 = kp.n1;
  if (n1 == 0) return pc;
  const int64_t nbk = std::min<int64_t>(256, (n + 4095) / 4096);
  const int64_t slab = (n + nbk - 1) / nbk;
  const int np = n1 * n1;
  double* part = c->get<double>(S_PC_PART, (size_t)nbk * np);
  k_gram<<<(unsigned)nbk, 256, 0, c->stream>>>(b.F, n, n1, slab, part);
  SDGP_CHECK_LAUNCH();
  std::vector<double> hp((size_t)nbk * np);
  SDGP_HIP(hipMemcpyAsync(hp.data(), part, hp.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  std::vector<double> Si;
  lowrank_finish(pc, n, nbk, hp.data(), Si);
  double* dSi = c->get<double>(S_PC_SINV, np);
  SDGP_HIP(hipMemcpyAsync(dSi, Si.data(), np * sizeof(double), hipMemcpyHostToDevice, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  pc.Sinv = dSi;
  return pc;
}

std::vector<Precond> lowrank_precond_pop(Ctx* c, const Sorted& s, const std::vector<KParams>& kp,
                                         const double* F0, std::vector<std::string>* failed) {
  const int B = (int)kp.size();
  const int64_t n = s.n;
  const int n1 = B > 0 ? kp[0].n1 : 0;
  const int n1s = n1 > 0 ? n1 : 1;
  std::vector<Precond> pcs(B);
  failed->assign(B, std::string());
  for (int m = 0; m < B; ++m) {
    try {
      pcs[m] = lowrank_base(kp[m], n, F0 + (size_t)m * n * n1s);
    } catch (const Error& e) {
      (*failed)[m] = e.what();
    }
  }
  if (n1 == 0 || B == 0) return pcs;
  const int64_t nbk = std::min<int64_t>(256, (n + 4095) / 4096);
  const int64_t slab = (n + nbk - 1) / nbk;
  const int np = n1 * n1;
  double* part = c->get<double>(S_POP_GRAM, (size_t)B * nbk * np);
  k_gram<<<dim3((unsigned)nbk, 1, B), 256, 0, c->stream>>>(F0, n, n1, slab, part);
  SDGP_CHECK_LAUNCH();
  std::vector<double> hp((size_t)B * nbk * np);
  SDGP_HIP(hipMemcpyAsync(hp.data(), part, hp.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  std::vector<double> all((size_t)B * np), Si;
  for (int m = 0; m < B; ++m) {
    if (!(*failed)[m].empty()) continue;
    try {
      lowrank_finish(pcs[m], n, nbk, hp.data() + (size_t)m * nbk * np, Si);
      std::copy(Si.begin(), Si.end(), all.begin() + (size_t)m * np);
    } catch (const Error& e) {
      (*failed)[m] = e.what();
    }
  }
  double* dSi = c->get<double>(S_POP_SINV, all.size());
  SDGP_HIP(hipMemcpyAsync(dSi, all.data(), all.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  for (int m = 0; m < B; ++m) pcs[m].Sinv = dSi + (size_t)m * np;
  return pcs;
}


namespace {

// Lanczos quadrature of one column per workgroup.  The column's tridiagonal T
// (d, e) follows from its CG coefficients, d_k = 1/a_k + b_{k-1}/a_{k-1} and
// e_k = sqrt(b_k)/a_k, and
//   e_1^T ln(T) e_1 = int_R t [1/(1+t) - e_1^T (T + tI)^{-1} e_1] ds, t = exp(s),
// which is ln(theta) = int_0^inf [1/(1+t) - 1/(theta+t)] dt on the spectral
// measure of e_1.  The integrand is analytic in the strip |Im s| < pi (poles at
// s = ln(theta_j) + i pi), so the trapezoidal rule with step h converges like
// exp(-2 pi^2 / h); the tails decay like exp(-|s|) beyond the spectrum.
// e_1^T (T + tI)^{-1} e_1 is the continued fraction of the bottom-up pivots of
// T + tI.  Nodes are the workgroup's threads (about 210 + 2.5 ln(condition)).
// The extreme Ritz values, which bound the nodes, come from Sturm counts (signs
// of the LDL^T pivots of T - xI) at 159 points at once for each of the two,
// each round cutting the interval by 160.
// Every chain is serial in k, one division a step (about 0.1 us), so what counts
// is how many run at once: all nodes of all columns.  On the host (16 threads)
// the quadrature took 65 ms for the 2000 unit columns of a 2000-point exact
// evaluation, and 7 ms for 32 probes of 2600 steps.
constexpr int kSlqT = 320;                      // threads: 5 wavefronts
constexpr int kSlqH = kSlqT / 2;                // points per extreme Ritz value
constexpr int kSlqC = 1024;                     // steps staged in LDS at a time
__global__ __launch_bounds__(kSlqT) void k_slq(const double* __restrict__ ha, const double* __restrict__ hb, int R,
                                               const int32_t* __restrict__ iters, int cap, double* __restrict__ out) {
  __shared__ double sd[kSlqC], se2[kSlqC];      // d_k, e_k^2
  __shared__ double red[kSlqT];
  __shared__ double iv[4];                      // [lo, hi] of the smallest, of the largest Ritz value
  __shared__ int hit[2], bad;
  const int r = 1 + blockIdx.x, t = threadIdx.x;
  double* o = out + 3 * (int64_t)blockIdx.x;
  const int m = cap > 0 ? min(iters[r], cap) : iters[r];
  if (m <= 0) {                                 // uniform
    if (t == 0) {
      o[0] = 0.0;
      o[1] = INFINITY;
      o[2] = -INFINITY;
    }
    return;
  }
  auto d_of = [&](int k) {
    double v = 1.0 / ha[(int64_t)k * R + r];
    if (k > 0) v += hb[(int64_t)(k - 1) * R + r] / ha[(int64_t)(k - 1) * R + r];
    return v;
  };
  auto e_of = [&](int k) { return k + 1 < m ? sqrt(hb[(int64_t)k * R + r]) / ha[(int64_t)k * R + r] : 0.0; };
  const int nch = (m + kSlqC - 1) / kSlqC;
  int held = -1;                                // chunk in LDS (uniform)
  auto stage = [&](int ch) {
    if (ch == held) return;
    __syncthreads();
    for (int k = ch * kSlqC + t; k < min(m, (ch + 1) * kSlqC); k += kSlqT) {
      const double e = e_of(k);
      sd[k - ch * kSlqC] = d_of(k);
      se2[k - ch * kSlqC] = e * e;
    }
    held = ch;
    __syncthreads();
  };
  // Gershgorin interval
  double glo = INFINITY, ghi = -INFINITY;
  int nan = 0;
  for (int k = t; k < m; k += kSlqT) {
    const double d = d_of(k), rr = (k > 0 ? fabs(e_of(k - 1)) : 0.0) + fabs(e_of(k));
    if (!isfinite(d) || !isfinite(rr)) nan = 1;
    glo = fmin(glo, d - rr);
    ghi = fmax(ghi, d + rr);
  }
  auto block_min = [&](double v) {
    red[t] = v;
    __syncthreads();
    if (t < 64) red[t] = fmin(fmin(fmin(red[t], red[t + 64]), fmin(red[t + 128], red[t + 192])), red[t + 256]);
    __syncthreads();
    if (t == 0)
      for (int k = 1; k < 64; ++k) red[0] = fmin(red[0], red[k]);
    __syncthreads();
    const double x = red[0];
    __syncthreads();
    return x;
  };
  if (t == 0) bad = 0;
  glo = block_min(glo);
  ghi = -block_min(-ghi);
  if (nan) bad = 1;
  __syncthreads();
  if (bad || !(ghi > 0.0) || !isfinite(glo) || !isfinite(ghi)) {
    if (t == 0) {
      o[0] = NAN;
      o[1] = o[2] = 0.0;
    }
    return;
  }
  // pivots of T - xI below zero
  auto sturm = [&](double x) {
    int cnt = 0;
    double q = 1.0, ep = 0.0;                   // first step: d_0 - x
    for (int ch = 0; ch < nch; ++ch) {
      stage(ch);
      const int e = min(m - ch * kSlqC, kSlqC);
      for (int k = 0; k < e; ++k) {
        if (q == 0.0) q = 1e-300;
        q = sd[k] - x - ep / q;
        ep = se2[k];
        if (q < 0.0) ++cnt;
      }
    }
    return cnt;
  };
  if (t == 0) {
    iv[0] = iv[2] = fmax(glo, 0.0);
    iv[1] = iv[3] = ghi;
  }
  __syncthreads();
  // point i of a half at the (i + 1)/160 part of its interval; the last of each
  // half, whose point would be the interval's end, counts at 0 instead (some
  // theta <= 0: no logarithm)
  for (int round = 0; round < 64; ++round) {
    const double a0 = iv[0], b0 = iv[1], a1 = iv[2], b1 = iv[3];
    const bool go = b0 - a0 > 1e-10 * b0 || b1 - a1 > 1e-10 * b1;
    if (!go && round > 0) break;
    const int half = t >= kSlqH ? 1 : 0, i = t - half * kSlqH;
    const double a = half ? a1 : a0, b = half ? b1 : b0;
    const bool zero = i == kSlqH - 1;
    const double x = zero ? 0.0 : a + (b - a) * ((i + 1) / (double)kSlqH);
    __syncthreads();                            // iv is read
    if (t < 2) hit[t] = kSlqH;
    const int cnt = sturm(x);
    __syncthreads();
    if (zero) {
      if (cnt != 0) bad = 1;
    } else if (cnt >= (half ? m : 1)) {
      atomicMin(&hit[half], i);
    }
    __syncthreads();
    if (bad) {
      if (t == 0) {
        o[0] = NAN;
        o[1] = o[2] = 0.0;
      }
      return;
    }
    if (t < 2) {
      const double la = t ? a1 : a0, lb = t ? b1 : b0;
      const int h = hit[t];                     // first point at or above the Ritz value
      if (h < kSlqH - 1) iv[2 * t + 1] = la + (lb - la) * ((h + 1) / (double)kSlqH);
      const int below = h < kSlqH ? h : kSlqH - 1;
      if (below > 0) iv[2 * t] = la + (lb - la) * (below / (double)kSlqH);
    }
    __syncthreads();
  }
  const double tmin = iv[1], tmax = iv[3];
  if (!(tmin > 0.0)) {
    if (t == 0) {
      o[0] = NAN;
      o[1] = tmin;
      o[2] = tmax;
    }
    return;
  }
  const double h = 0.4;
  const double s0 = log(tmin) - 42.0, s1 = log(tmax) + 42.0;
  const int nodes = (int)ceil((s1 - s0) / h);
  double acc = 0.0;
  for (int j0 = 0; j0 <= nodes; j0 += kSlqT) {
    const int j = j0 + t;
    const double x = exp(s0 + min(j, nodes) * h);
    double f = 1.0;
    for (int ch = nch - 1; ch >= 0; --ch) {
      stage(ch);
      int k = min(m - ch * kSlqC, kSlqC) - 1;
      if (ch == nch - 1) {
        f = sd[k] + x;
        --k;
      }
      for (; k >= 0; --k) f = sd[k] + x - se2[k] / f;
    }
    if (j <= nodes) acc += x * (1.0 / (1.0 + x) - 1.0 / f);
  }
  __syncthreads();
  red[t] = acc;
  __syncthreads();
  if (t < 64) red[t] = ((red[t] + red[t + 64]) + (red[t + 128] + red[t + 192])) + red[t + 256];
  __syncthreads();
  if (t < 64) {
    const double s = wave_sum(red[t]);
    if (t == 0) {
      o[0] = h * s;
      o[1] = tmin;
      o[2] = tmax;
    }
  }
}

}  // namespace

void slq_from_cg(Ctx* c, const CgResult& cg, int kind, int P, int64_t n, int lanczos_steps, double* logdet,
                 double* stderr_out, double* ritz_min, double* ritz_max) {
  (void)P;
  (void)n;
  const int ncols = cg.R - 1;
  if (ncols <= 0) {
    *logdet = 0.0; *stderr_out = 0.0; *ritz_min = 0.0; *ritz_max = 0.0;
    return;
  }
  double* dq = c->get<double>(S_SLQ_OUT, (size_t)ncols * 3);
  k_slq<<<(unsigned)ncols, kSlqT, 0, c->stream>>>(cg.hist_a, cg.hist_b, cg.R, cg.col_iters, lanczos_steps, dq);
  SDGP_CHECK_LAUNCH();
  std::vector<double> w0(cg.R), qlh((size_t)ncols * 3);   // (quadrature, smallest, largest Ritz value) per column
  SDGP_HIP(hipMemcpyAsync(w0.data(), cg.rz0, cg.R * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipMemcpyAsync(qlh.data(), dq, qlh.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  // weight of probe p: |M^{-1/2} b_p|^2 = b_p^T M^{-1} b_p (|z|^2 without a
  // preconditioner: n for Rademacher, 1 for unit vectors)
  double sum = 0.0, sum2 = 0.0, mn = INFINITY, mx = -INFINITY;
  bool bad = false;
  for (int p = 0; p < ncols; ++p) {
    const double v = w0[1 + p] * qlh[3 * p];
    if (!std::isfinite(v)) bad = true;
    sum += v;
    sum2 += v * v;
    mn = std::min(mn, qlh[3 * p + 1]);
    mx = std::max(mx, qlh[3 * p + 2]);
  }
  if (bad) throw Error(SDGP_ERR_NOT_SPD, "Lanczos quadrature met a non-positive Ritz value");
  if (kind == PK_IDENTITY) {
    *logdet = cg.logdetM + sum;
    *stderr_out = 0.0;
  } else {
    const double mean = sum / ncols;
    *logdet = cg.logdetM + mean;
    const double var = ncols > 1 ? std::max(0.0, (sum2 - ncols * mean * mean) / (ncols - 1)) : 0.0;
    *stderr_out = ncols > 1 ? std::sqrt(var / ncols) : NAN;
  }
  *ritz_min = mn;
  *ritz_max = mx;
}

}  // namespace sdgp
