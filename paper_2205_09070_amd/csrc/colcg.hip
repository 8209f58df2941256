// Column conjugate gradients (Section 2.5) for small point sets on gfx950.
//
// The columns of the block CG are independent, and below about ten thousand
// points a column's search direction fits in one CU's LDS.  Here one workgroup
// runs the whole solve of 1, 2 or 4 columns in a single launch: p lives in
// LDS, r and A p in registers (row by row of a thread), x in memory, and the
// only synchronisation is the workgroup's barrier, where the block CG pays
// five to eight launches and two grid-wide reductions per iteration.  What a
// solve then costs per iteration is its read of the matrix (10 B per entry,
// from the L2) and one LDS gather per entry and column.
//
// Matrix layout: rows sorted by length (longest first), 64 rows per slice and
// wavefront, four entries of a row at a time: a slice step is 64 x 4 values
// (two 16-byte loads per lane) and 64 x 4 16-bit places (one 8-byte load), so
// every load is contiguous over the wavefront and the slices' padding stays
// small.  Vectors are indexed by the row's place in that order.
//
// Iterations, stopping, failure and the recorded coefficients are those of the
// block CG (cg.hip); sums run in a fixed order.
#include <algorithm>
#include <cmath>
#include <vector>

#include "kernel_math.hpp"
#include "sdgp_internal.hpp"

namespace sdgp {

namespace {

// The kernels read their arrays through pointers held in device memory, which
// the compiler cannot prove to be global; this type lets it emit global (not
// flat) memory instructions, which also leave the LDS counter alone.
#define GL __attribute__((address_space(1)))
typedef double dv2 __attribute__((ext_vector_type(2)));
typedef uint32_t uv2 __attribute__((ext_vector_type(2)));

struct ColArgs {
  int64_t n;
  int npad, S, R, n1;
  int use_pc, lowrank_op, max_iter, kind;
  uint64_t seed;
  double inv_c, sqrt_c, rtol2, prtol2;
  const int64_t* row_ptr;
  const int32_t* csr_col;
  const double* csr_val;
  const double* F;          // [n][n1] sorted bump values
  int32_t* order;           // place -> row
  int32_t* place;           // row -> place
  int32_t* width;           // [S] slice steps
  int64_t* off;             // [S] first step
  dv2* val;                 // [step][2][64]
  uv2* col;                 // [step][64], four 16-bit places each
  double* FT;               // [n1][npad] bump values by place
  const double* Sinv;
  const double* ys;
  const int32_t* perm;
  const double* dense;
  double *X, *V;            // [n][R] (V: M^{-1} b, may be null)
  double* xw;               // [R][npad] x by place
  double *hist_a, *hist_b;  // [max_iter][R] (null: not kept)
  double *rz0, *bn, *rl;    // [R]
  int32_t *iters, *flags;   // [R] (flags: 1 failed, 2 still iterating at max_iter)
  int none;                 // 0 (see slice_of in k_col_cg)
};

// Place of every row: rows by descending length, equal ones by index, i.e. the
// number of rows ahead of it (n is at most kColMaxN).  16 lanes per row.
__global__ __launch_bounds__(256) void k_col_rank(const ColArgs* __restrict__ AA) {
  const ColArgs& A = AA[blockIdx.y];
  const int n = (int)A.n;
  const int a = blockIdx.x * 16 + (threadIdx.x >> 4), part = threadIdx.x & 15;
  const GL int64_t* rp = (const GL int64_t*)A.row_ptr;
  const int mine = a < n ? (int)(rp[a + 1] - rp[a]) : -1;
  int rank = 0;
#pragma unroll 4
  for (int b = part; b < n; b += 16) {
    const int len = (int)(rp[b + 1] - rp[b]);
    rank += (len > mine || (len == mine && b < a)) ? 1 : 0;
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) rank += __shfl_xor(rank, o, 16);
  if (part != 0) return;
  if (a < n) {
    A.order[rank] = a;
    A.place[a] = rank;
  } else if (a < A.npad) {
    A.order[a] = -1;
  }
}

// Steps and first step of every slice (its first row is its longest).
__global__ __launch_bounds__(64) void k_col_slices(const ColArgs* __restrict__ AA) {
  const ColArgs& A = AA[blockIdx.x];
  const int lane = threadIdx.x;
  int64_t base = 0;
  for (int s0 = 0; s0 < A.S; s0 += 64) {
    const int s = s0 + lane;
    int w = 0;
    if (s < A.S) {
      const int a = A.order[64 * s];
      w = (int)((A.row_ptr[a + 1] - A.row_ptr[a] + 3) >> 2);
    }
    int incl = w;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o, 64);
      if (lane >= o) incl += u;
    }
    if (s < A.S) {
      A.width[s] = w;
      A.off[s] = base + incl - w;
    }
    base += readlane_i32(incl, 63);
  }
}

// The slice's entries (one row per lane, the steps dealt to the block's
// wavefronts; places past a row's end hold 0 at the row's own place), and its
// part of F by place.
__global__ __launch_bounds__(512) void k_col_fill(const ColArgs* __restrict__ AA) {
  const ColArgs& A = AA[blockIdx.y];
  const int s = blockIdx.x, lane = lane_id(), wv = threadIdx.x >> 6;
  const int pos = 64 * s + lane;
  const int a = ((const GL int32_t*)A.order)[pos];
  const GL int64_t* rp = (const GL int64_t*)A.row_ptr;
  const GL int32_t* cc = (const GL int32_t*)A.csr_col;
  const GL double* cv = (const GL double*)A.csr_val;
  const GL int32_t* place = (const GL int32_t*)A.place;
  const int64_t k0 = a >= 0 ? rp[a] : 0, e = a >= 0 ? rp[a + 1] : 0;
  const int w = ((const GL int32_t*)A.width)[s];
  const int64_t base = ((const GL int64_t*)A.off)[s];
  const uint32_t self = (uint32_t)pos;
  for (int t = wv; t < w; t += 8) {
    const int64_t k = k0 + 4 * t;
    double v[4];
    int32_t b[4];
    uint32_t c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[u] = k + u < e ? cv[k + u] : 0.0;
      b[u] = k + u < e ? cc[k + u] : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) c[u] = b[u] >= 0 ? (uint32_t)place[b[u]] : self;
    ((GL dv2*)A.val)[((base + t) * 2 + 0) * 64 + lane] = dv2{v[0], v[1]};
    ((GL dv2*)A.val)[((base + t) * 2 + 1) * 64 + lane] = dv2{v[2], v[3]};
    ((GL uv2*)A.col)[(base + t) * 64 + lane] = uv2{c[0] | c[1] << 16, c[2] | c[3] << 16};
  }
  for (int i = wv; i < A.n1; i += 8)
    ((GL double*)A.FT)[(int64_t)i * A.npad + pos] = a >= 0 ? ((const GL double*)A.F)[(int64_t)a * A.n1 + i] : 0.0;
}

// Right-hand sides by place (as k_cg_start of the block CG) into x's storage.
__global__ __launch_bounds__(256) void k_col_rhs(const ColArgs* __restrict__ AA) {
  const ColArgs& A = AA[blockIdx.z];
  const int pos = blockIdx.x * 256 + threadIdx.x, rc = blockIdx.y;
  if (pos >= A.npad) return;
  const int a = A.order[pos];
  double b = 0.0;
  if (a >= 0) {
    if (A.kind == PK_DENSE) {
      b = A.dense[(int64_t)a * A.R + rc];
    } else if (rc == 0) {
      b = A.ys[a];
    } else if (A.kind == PK_IDENTITY) {
      b = A.perm[a] == rc - 1 ? 1.0 : 0.0;
    } else {
      const uint64_t pbase = (uint64_t)(rc - 1) << 32;
      b = (splitmix64_at(A.seed, pbase + (uint64_t)A.perm[a] + 1ull) >> 63) ? -1.0 : 1.0;
      if (A.use_pc) {
        double fv = 0.0;
        for (int i = 0; i < A.n1; ++i) {
          const double v = (splitmix64_at(A.seed, pbase + 0xFFFFFFFFull - (uint64_t)i) >> 63) ? -1.0 : 1.0;
          fv += A.F[(int64_t)a * A.n1 + i] * v;
        }
        b = A.sqrt_c * b + fv;
      }
    }
  }
  A.xw[(int64_t)rc * A.npad + pos] = b;
}

// Sum over the wavefront, the same in every lane: within each 16-lane row by
// DPP rotations, then the four rows in order.
template <int ctrl>
__device__ __forceinline__ double dpp_d(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), ctrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double wave_total(double v) {
  v += dpp_d<0x128>(v);   // row_ror 8, 4, 2, 1
  v += dpp_d<0x124>(v);
  v += dpp_d<0x122>(v);
  v += dpp_d<0x121>(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// Four entries of the lane's row: acc += their products with p (LDS).
template <int NC>
__device__ __forceinline__ void col_step(const dv2& v01, const dv2& v23, const uv2& c, const double* p, double* acc) {
  const uint32_t at[4] = {c.x & 0xffffu, c.x >> 16, c.y & 0xffffu, c.y >> 16};
  const double v[4] = {v01.x, v01.y, v23.x, v23.y};
  double x[4][NC];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if constexpr (NC == 1) {
      x[u][0] = p[at[u]];
    } else {
#pragma unroll
      for (int h = 0; h < NC; h += 2) {
        const dv2 t = *reinterpret_cast<const dv2*>(p + at[u] * NC + h);
        x[u][h] = t.x;
        x[u][h + 1] = t.y;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[q] += v[u] * x[u][q];
}

// Workgroup barrier that orders LDS only.  What the solve's threads write to
// memory (x, the coefficients) is read by nobody until the kernel ends, and a
// full barrier would wait for those stores at every reduction: an iteration
// of a 2,000-point solve took 10.4 us with it and with generic (flat) memory
// instructions, 9.4 us with this one and global ones.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Columns NC blockIdx.x .. of member blockIdx.y.  W wavefronts, each holding
// the vectors of RPT slices (dealt in turn there and back, which evens out
// their lengths); kRows: rows that p's LDS holds; kF: preconditioner and / or
// F F^T operator.
template <int W, int RPT, int NC, int kRows, bool kF>
__global__ __launch_bounds__(64 * W) void k_col_cg(const ColArgs* __restrict__ AA) {
  const ColArgs& A = AA[blockIdx.y];
  constexpr int U = RPT * NC > 8 ? 2 : 4;        // slice steps loaded together
  __shared__ __align__(16) double p[kRows * NC];
  __shared__ double red[2][NC * W];
  __shared__ double redF[kF ? kMaxN1 * NC * W : 1];
  __shared__ double sg[kF ? kMaxN1 * NC : 1], su[kF ? kMaxN1 * NC : 1];
  __shared__ int soff[kRows / 64 + 1];           // first step of every slice, all steps
  constexpr bool kXR = RPT * NC <= 8;            // x in registers (else by place in memory)
  const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int R = A.R, S = A.S, n1 = A.n1, npad = A.npad;
  const bool pc = kF && A.use_pc, lr = kF && A.lowrank_op;
  const int rc0 = blockIdx.x * NC;
  const GL int32_t* order = (const GL int32_t*)A.order;
  const GL double* FT = (const GL double*)A.FT;
  GL double* xw = (GL double*)A.xw;
  GL double* Vo = (GL double*)A.V;
  // slice k of the wavefront, -1 past the last.  turn is 0, in a way that the
  // compiler has to work out in every iteration: it would otherwise compute
  // every slice's addresses ahead of the solve and spill them.
  int turn = 0;
  auto slice_of = [&](int k) {
    const int s = __builtin_amdgcn_readfirstlane(k * W + ((k & 1) ? W - 1 - w : w) + turn);
    return s < S ? s : -1;
  };
  for (int sl = threadIdx.x; sl <= S; sl += 64 * W) {
    const int k = min(sl, S - 1);
    soff[sl] = (int)((const GL int64_t*)A.off)[k] + (sl > k ? ((const GL int32_t*)A.width)[k] : 0);
  }
  lds_barrier();
  int phase = 0;
  // sums of NC values over the workgroup, the same in every thread
  auto block_total = [&](double* v) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const double t = wave_total(v[q]);
      if (lane == 0) red[phase][q * W + w] = t;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < W; ++k) t += red[phase][q * W + k];
      v[q] = t;
    }
    phase ^= 1;
  };
  // F^T v of the register vectors into dst (LDS, [i][NC]) after a barrier
  auto ft_parts = [&](const double (&v)[RPT][NC]) {
    for (int i = 0; i < n1; ++i) {
      double t[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) t[q] = 0.0;
#pragma unroll
      for (int k = 0; k < RPT; ++k)
        if (const int sl = slice_of(k); sl >= 0) {
          const double f = FT[(int64_t)i * npad + 64 * sl + lane];
#pragma unroll
          for (int q = 0; q < NC; ++q) t[q] += f * v[k][q];
        }
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const double s = wave_total(t[q]);
        if (lane == 0) redF[(i * NC + q) * W + w] = s;
      }
    }
  };
  auto ft_total = [&](double* dst) {
    for (int t = threadIdx.x; t < n1 * NC; t += 64 * W) {
      double s = 0.0;
#pragma unroll
      for (int k = 0; k < W; ++k) s += redF[t * W + k];
      dst[t] = s;
    }
  };
  // u = S^{-1} g into su, and g.u
  auto small_solve = [&](double* gu) {
    for (int t = threadIdx.x; t < n1 * NC; t += 64 * W) {
      const int i = t / NC, q = t - i * NC;
      double s = 0.0;
      for (int k = 0; k < n1; ++k) s += ((const GL double*)A.Sinv)[i * n1 + k] * sg[k * NC + q];
      su[t] = s;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < NC; ++q) gu[q] = 0.0;
    for (int k = 0; k < n1; ++k)
#pragma unroll
      for (int q = 0; q < NC; ++q) gu[q] += sg[k * NC + q] * su[k * NC + q];
  };
  // sum_i F[row][i] c[i] of the thread's row in slice s
  auto f_dot = [&](int s, const double* c, double* out) {
#pragma unroll
    for (int q = 0; q < NC; ++q) out[q] = 0.0;
    for (int i = 0; i < n1; ++i) {
      const double f = FT[(int64_t)i * npad + 64 * s + lane];
#pragma unroll
      for (int q = 0; q < NC; ++q) out[q] += f * c[i * NC + q];
    }
  };

  // acc += the products of the lane's row in the slice of e steps at step base
  auto steps = [&](int64_t base, int e, double* acc) {
    // uniform base and 32-bit lane offsets (a slice's storage is below 4 GiB)
    const GL char *vb = (const GL char*)(A.val + base * 128), *cb = (const GL char*)(A.col + base * 64);
    auto val_at = [&](int i, int h) {
      return *(const GL dv2*)(vb + ((uint32_t)(2 * i + h) * 1024u + (uint32_t)lane * 16u));
    };
    auto col_at = [&](int i) { return *(const GL uv2*)(cb + ((uint32_t)i * 512u + (uint32_t)lane * 8u)); };
    int t = 0;
    for (; t + U <= e; t += U) {
      dv2 v0[U], v1[U];
      uv2 c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v0[u] = val_at(t + u, 0);
        v1[u] = val_at(t + u, 1);
        c[u] = col_at(t + u);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) col_step<NC>(v0[u], v1[u], c[u], p, acc);
    }
    for (; t < e; ++t) col_step<NC>(val_at(t, 0), val_at(t, 1), col_at(t), p, acc);
  };

  // right-hand sides (left in x's storage by k_col_rhs), x = 0
  double r[RPT][NC], qv[RPT][NC], x[kXR ? RPT : 1][NC];
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      r[k][q] = 0.0;
      if constexpr (kXR) x[k][q] = 0.0;
    }
    const int sl = slice_of(k);
    if (sl < 0) continue;
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (rc0 + q < R) {
        GL double* xp = xw + (int64_t)(rc0 + q) * npad + 64 * sl + lane;
        r[k][q] = *xp;
        if constexpr (!kXR) *xp = 0.0;
      }
  }
  double bb[NC], rz[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    bb[q] = 0.0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) bb[q] += r[k][q] * r[k][q];
  }
  if (pc) ft_parts(r);
  block_total(bb);
#pragma unroll
  for (int q = 0; q < NC; ++q) rz[q] = bb[q];
  if (pc) {
    double gu[NC];
    ft_total(sg);
    lds_barrier();
    small_solve(gu);
#pragma unroll
    for (int q = 0; q < NC; ++q) rz[q] = (bb[q] - gu[q]) * A.inv_c;
  }
  // p = z0; V = z0
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int sl = slice_of(k);
    if (sl < 0) continue;
    double z[NC], u[NC];
    if (pc) f_dot(sl, su, u);
    const int pos = 64 * sl + lane;
    const int a = order[pos];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      z[q] = pc ? (r[k][q] - u[q]) * A.inv_c : r[k][q];
      p[pos * NC + q] = z[q];
      if (Vo && a >= 0 && rc0 + q < R) Vo[(int64_t)a * R + rc0 + q] = z[q];
      qv[k][q] = z[q];
    }
  }
  if (lr) {
#pragma unroll
    for (int k = 0; k < RPT; ++k)
      if (slice_of(k) < 0)
#pragma unroll
        for (int q = 0; q < NC; ++q) qv[k][q] = 0.0;
    ft_parts(qv);
  }
  lds_barrier();
  if (lr) {
    ft_total(sg);
    lds_barrier();
  }
  bool act[NC], failed[NC];
  int its[NC];
  double rl[NC];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    act[q] = rc0 + q < R && bb[q] > 0.0;
    failed[q] = false;
    its[q] = 0;
    rl[q] = bb[q];
  }
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (rc0 + q < R) {
        ((GL double*)A.rz0)[rc0 + q] = rz[q];
        ((GL double*)A.bn)[rc0 + q] = bb[q];
      }
  const int none = A.none;
  for (int it = 0; it < A.max_iter; ++it) {
    turn = it & none;
    bool any = false;
#pragma unroll
    for (int q = 0; q < NC; ++q) any |= act[q];
    if (!any) break;
    // A p, and p.A p
    double d[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) d[q] = 0.0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      double acc[NC];
#pragma unroll
      for (int q = 0; q < NC; ++q) acc[q] = 0.0;
      if (const int sl = slice_of(k); sl >= 0) {
        const int so = __builtin_amdgcn_readfirstlane(soff[sl]);
        steps(so, __builtin_amdgcn_readfirstlane(soff[sl + 1]) - so, acc);
        double f[NC];
        if (lr) f_dot(sl, sg, f);
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          d[q] += p[(64 * sl + lane) * NC + q] * acc[q];
          if (lr) acc[q] += f[q];
        }
      }
#pragma unroll
      for (int q = 0; q < NC; ++q) qv[k][q] = acc[q];
    }
    block_total(d);
    if (lr)
      for (int i = 0; i < n1; ++i)
#pragma unroll
        for (int q = 0; q < NC; ++q) d[q] += sg[i * NC + q] * sg[i * NC + q];
    double alpha[NC], rr[NC];
    bool upd[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      alpha[q] = 0.0;
      upd[q] = false;
      if (act[q]) {
        if (d[q] > 0.0 && isfinite(d[q])) {
          alpha[q] = rz[q] / d[q];
          upd[q] = true;
        } else {
          failed[q] = true;
          act[q] = false;
        }
        if (threadIdx.x == 0 && A.hist_a) ((GL double*)A.hist_a)[(int64_t)it * R + rc0 + q] = alpha[q];
      }
      rr[q] = 0.0;
    }
    // x += alpha p, r -= alpha A p
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int sl = slice_of(k);
    if (sl < 0) continue;
      const int pos = 64 * sl + lane;
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        if (upd[q]) {
          if constexpr (kXR) x[k][q] += alpha[q] * p[pos * NC + q];
          else xw[(int64_t)(rc0 + q) * npad + pos] += alpha[q] * p[pos * NC + q];
          r[k][q] -= alpha[q] * qv[k][q];
        }
        rr[q] += r[k][q] * r[k][q];
      }
    }
    if (pc) ft_parts(r);
    block_total(rr);
    double zz[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) zz[q] = rr[q];
    if (pc) {
      double gu[NC];
      ft_total(sg);
      lds_barrier();
      small_solve(gu);
#pragma unroll
      for (int q = 0; q < NC; ++q) zz[q] = (rr[q] - gu[q]) * A.inv_c;
    }
    double beta[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      beta[q] = 0.0;
      if (upd[q]) {
        beta[q] = zz[q] / rz[q];
        rz[q] = zz[q];
        rl[q] = rr[q];
        ++its[q];
        act[q] = !(rr[q] <= (rc0 + q == 0 ? A.rtol2 : A.prtol2) * bb[q]);
        if (threadIdx.x == 0 && A.hist_a) ((GL double*)A.hist_b)[(int64_t)it * R + rc0 + q] = beta[q];
      }
    }
    // p = M^{-1} r + beta p
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int sl = slice_of(k);
    if (sl < 0) continue;
      const int pos = 64 * sl + lane;
      double u[NC];
      if (pc) f_dot(sl, su, u);
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        const double z = pc ? (r[k][q] - u[q]) * A.inv_c : r[k][q];
        const double pn = act[q] ? z + beta[q] * p[pos * NC + q] : p[pos * NC + q];
        p[pos * NC + q] = pn;
        if (lr) qv[k][q] = pn;
      }
    }
    if (lr) ft_parts(qv);
    lds_barrier();
    if (lr) {
      ft_total(sg);
      lds_barrier();
    }
  }
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (rc0 + q < R) {
        ((GL double*)A.rl)[rc0 + q] = rl[q];
        ((GL int32_t*)A.iters)[rc0 + q] = its[q];
        ((GL int32_t*)A.flags)[rc0 + q] = (failed[q] ? 1 : 0) | (act[q] ? 2 : 0);
      }
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int sl = slice_of(k);
    if (sl < 0) continue;
    const int pos = 64 * sl + lane;
    const int a = order[pos];
    if (a < 0) continue;
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (rc0 + q < R) ((GL double*)A.X)[(int64_t)a * R + rc0 + q] = kXR ? x[kXR ? k : 0][q] : xw[(int64_t)(rc0 + q) * npad + pos];
  }
}

constexpr int kColMaxN = 10048;      // rows of p that fit in LDS twice (157 slices of 64)

// Columns per workgroup for n rows and R columns (see column_cg).
int columns_per_group(int64_t n, int R, bool f) {
  if (R <= 256) return 1;
  if (n <= 2048) return 4;
  return (n <= 4096 || !f) ? 2 : 1;
}

template <bool kF>
void launch_col(hipStream_t st, const ColArgs* dA, int64_t n, int R, int NC, int B) {
  const dim3 g((unsigned)((R + NC - 1) / NC), (unsigned)B);
  if (n <= 2048) {
    if (NC == 1) k_col_cg<16, 2, 1, 2048, kF><<<g, 1024, 0, st>>>(dA);
    else k_col_cg<8, 4, 4, 2048, kF><<<g, 512, 0, st>>>(dA);
  } else if (n <= 4096) {
    if (NC == 1) k_col_cg<16, 4, 1, 4096, kF><<<g, 1024, 0, st>>>(dA);
    else k_col_cg<16, 4, 2, 4096, kF><<<g, 1024, 0, st>>>(dA);
  } else if (NC == 1) {
    k_col_cg<16, 10, 1, kColMaxN, kF><<<g, 1024, 0, st>>>(dA);
  } else {
    if constexpr (!kF) k_col_cg<16, 10, 2, kColMaxN, false><<<g, 1024, 0, st>>>(dA);
  }
  SDGP_CHECK_LAUNCH();
}

// Slice steps that a member's matrix can take: every slice but the first is as
// wide as some row ahead of it, so its padding fits in that row's slice.
int64_t max_steps(int64_t n, int64_t nnz) { return nnz / 256 + 2 * ((n + 63) / 64) + (n + 3) / 4 + 1; }

}  // namespace

// Column CG or block CG, by the time of one iteration of a single solve (us),
// from measurements at 64 .. 10,000 points.  Column CG: 2.5 us of reductions
// and the matrix's 10 B per entry at 130 GB/s per CU (64 GB/s when most CUs
// stream it), F read four times, in as many rounds as the CUs need for the
// columns; block CG: 40 us of launches, and per slab of 32 columns the gathers
// at 15 TB/s and eight vector passes at 4 TB/s.  (2,000 points in the plane, 37
// entries per row, 33 columns: 9.4 against 36 us; its 2,001 columns for the
// exact likelihood: 28 against 213 us; 10,000 points, 88 entries per row, 501
// columns: 137 us against eight solves of about 90 us.)  A population's members
// are taken as single solves here, so that both give the same values; that the
// block CG shares its launches among members does not enter.
bool column_cg_applies(const Ctx* c, int64_t n, int64_t nnz, int R, int n1, bool keep_v, int max_iter) {
  if (n > kColMaxN || nnz < 0) return false;
  const int NC = columns_per_group(n, R, n1 > 0);
  const int64_t groups = (R + NC - 1) / NC, cu = std::max(1, c->cu_count), ns = (R - 1 + 31) / 32;
  const double rate = 2 * groups > cu ? 64e3 : 130e3;            // bytes per us and CU
  const double col_us = (double)((groups + cu - 1) / cu) * (2.5 + (10.0 * nnz + 32.0 * n1 * n) / rate);
  const double block_us = 40.0 + ns * (256.0 * nnz / 15e6 + 2048.0 * n / 4e6);
  if (col_us > block_us) return false;
  // Limited workspace.  A context under a cap keeps to the block CG: the column
  // CG holds buffers of its own (the matrix in slices) beside those that the
  // block CG needs for other sizes, and what fitted the cap without it has to fit
  // in any order of calls.  The static workspace starts empty at every call, so
  // there the sizes decide: column CG where it leaves half of the room to the
  // quadrature and the adjoint, or takes no more than the block CG's vectors and
  // coefficients.
  if (!c->arena) return c->cap_bytes == 0;
  const int64_t npad = (n + 63) / 64 * 64;
  const double hist = 16.0 * max_iter * R;
  const double need = 8.0 * R * ((keep_v ? 2.0 : 1.0) * n + npad) + 2560.0 * max_steps(n, nnz) + 8.0 * n1 * npad +
                      hist + 9.0 * npad + 32.0 * R + 4096.0;
  const double block_need = 8.0 * (keep_v ? 5.0 : 4.0) * (n + 32.0 * ns * n) + hist;
  return 2.25 * need <= (double)(c->arena_cap - c->arena_used) || need <= block_need;
}

std::vector<CgResult> column_cg(Ctx* c, const std::vector<CgMember>& mem, const Sorted& s, const double* ys, int kind,
                                int R, uint64_t seed, double rtol, double prtol, int max_iter,
                                const double* dense_rhs, bool keep_v, bool beside) {
  const int B = (int)mem.size();
  const int64_t n = s.n;
  const int S = (int)((n + 63) / 64), npad = 64 * S;
  const Precond* pc0 = mem[0].pc;
  const bool use_pc = pc0 != nullptr && pc0->n1 > 0 && pc0->apply;
  const bool use_lr = pc0 != nullptr && pc0->n1 > 0 && pc0->lowrank_op;
  const bool f = use_pc || use_lr;
  const int n1 = f ? pc0->n1 : 0;
  const int NC = columns_per_group(n, R, f);
  std::vector<int64_t> soff(B + 1, 0);
  for (int m = 0; m < B; ++m) soff[m + 1] = soff[m] + max_steps(n, mem[m].A.nnz);
  const size_t NR = (size_t)n * R;
  // (the block CG's results lie in P, Q, the state and the histories; its X, R
  // and V are working storage)
  double* X = c->get<double>(beside ? S_CG_R : S_CG_P, NR * B);
  double* V = (use_pc && keep_v) ? c->get<double>(beside ? S_CG_V : S_CG_Q, NR * B) : nullptr;
  double* xw = c->get<double>(S_CG_X, (size_t)npad * R * B);
  int32_t* idx = c->get<int32_t>(S_COL_IDX, (size_t)(2 * npad + S) * B);
  int64_t* off = c->get<int64_t>(S_COL_OFF, (size_t)S * B);
  dv2* val = c->get<dv2>(S_COL_VAL, (size_t)soff[B] * 128);
  uv2* col = c->get<uv2>(S_COL_COL, (size_t)soff[B] * 64);
  double* FT = n1 > 0 ? c->get<double>(S_COL_FT, (size_t)n1 * npad * B) : nullptr;
  // the coefficients are read by the quadrature of probe columns only
  const bool keep_hist = kind == PK_RADEMACHER || kind == PK_IDENTITY;
  double* ha = keep_hist ? c->get<double>(beside ? S_COL_HIST_A : S_CG_HIST_A, (size_t)max_iter * R * B) : nullptr;
  double* hb = keep_hist ? c->get<double>(beside ? S_COL_HIST_B : S_CG_HIST_B, (size_t)max_iter * R * B) : nullptr;
  double* sd = c->get<double>(S_COL_STATE, (size_t)R * B * 3);          // rz0, bn, rl of every member
  int32_t* si = c->get<int32_t>(S_COL_ITERS, (size_t)R * B * 2);        // iters, flags
  std::vector<ColArgs> hA(B);
  for (int m = 0; m < B; ++m) {
    ColArgs& A = hA[m];
    const Precond* p = mem[m].pc;
    A.n = n; A.npad = npad; A.S = S; A.R = R; A.n1 = n1;
    A.use_pc = use_pc ? 1 : 0; A.lowrank_op = use_lr ? 1 : 0; A.max_iter = max_iter; A.kind = kind; A.seed = seed;
    A.inv_c = use_pc ? 1.0 / p->c : 1.0;
    A.sqrt_c = use_pc ? std::sqrt(p->c) : 1.0;
    A.rtol2 = rtol * rtol; A.prtol2 = prtol * prtol;
    A.row_ptr = mem[m].A.row_ptr; A.csr_col = mem[m].A.col; A.csr_val = mem[m].A.val;
    A.F = n1 > 0 ? p->F : nullptr;
    A.order = idx + (size_t)m * (2 * npad + S);
    A.place = A.order + npad;
    A.width = A.place + npad;
    A.off = off + (size_t)m * S;
    A.val = val + soff[m] * 128;
    A.col = col + soff[m] * 64;
    A.FT = n1 > 0 ? FT + (size_t)m * n1 * npad : nullptr;
    A.Sinv = use_pc ? p->Sinv : nullptr;
    A.ys = ys; A.perm = s.perm; A.dense = dense_rhs;
    A.X = X + m * NR;
    A.V = V ? V + m * NR : nullptr;
    A.xw = xw + (size_t)m * npad * R;
    A.hist_a = keep_hist ? ha + (size_t)m * max_iter * R : nullptr;
    A.hist_b = keep_hist ? hb + (size_t)m * max_iter * R : nullptr;
    A.rz0 = sd + (size_t)m * R * 3;
    A.bn = A.rz0 + R;
    A.rl = A.bn + R;
    A.iters = si + (size_t)m * R * 2;
    A.flags = A.iters + R;
    A.none = 0;
  }
  ColArgs* dA = c->get<ColArgs>(S_CG_ARGS, B);
  SDGP_HIP(hipMemcpyAsync(dA, hA.data(), B * sizeof(ColArgs), hipMemcpyHostToDevice, c->stream));
  k_col_rank<<<dim3((unsigned)(npad / 16), (unsigned)B), 256, 0, c->stream>>>(dA);
  SDGP_CHECK_LAUNCH();
  k_col_slices<<<(unsigned)B, 64, 0, c->stream>>>(dA);
  SDGP_CHECK_LAUNCH();
  k_col_fill<<<dim3((unsigned)S, (unsigned)B), 512, 0, c->stream>>>(dA);
  SDGP_CHECK_LAUNCH();
  k_col_rhs<<<dim3((unsigned)((npad + 255) / 256), (unsigned)R, (unsigned)B), 256, 0, c->stream>>>(dA);
  SDGP_CHECK_LAUNCH();
  if (f) launch_col<true>(c->stream, dA, n, R, NC, B);
  else launch_col<false>(c->stream, dA, n, R, NC, B);
  std::vector<double> hd((size_t)R * B * 3);
  std::vector<int32_t> hi((size_t)R * B * 2);
  SDGP_HIP(hipMemcpyAsync(hd.data(), sd, hd.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipMemcpyAsync(hi.data(), si, hi.size() * sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
  SDGP_HIP(hipStreamSynchronize(c->stream));
  std::vector<CgResult> out(B);
  for (int m = 0; m < B; ++m) {
    CgResult& res = out[m];
    const ColArgs& A = hA[m];
    res.R = R;
    res.X = A.X;
    res.V = A.V;
    res.rz0 = A.rz0;
    res.hist_a = A.hist_a;
    res.hist_b = A.hist_b;
    res.col_iters = A.iters;
    res.logdetM = use_pc ? mem[m].pc->logdetM : 0.0;
    res.not_spd = false;
    bool running = false;
    int done = 1;                    // an iteration is counted also when no column had one
    res.relres_max = 0.0;
    for (int r = 0; r < R; ++r) {
      const int it = hi[(size_t)m * R * 2 + r], fl = hi[(size_t)m * R * 2 + R + r];
      done = std::max(done, it + (fl & 1));
      if (fl & 1) res.not_spd = true;
      if (fl & 2) running = true;
      const double b2 = hd[(size_t)m * R * 3 + R + r];
      if (b2 > 0.0) res.relres_max = std::max(res.relres_max, std::sqrt(hd[(size_t)m * R * 3 + 2 * R + r] / b2));
    }
    res.iters = done;
    res.iters_y = hi[(size_t)m * R * 2];
    res.converged = !running && !res.not_spd;
  }
  c->last_shape = TuneChoice();
  c->last_shape.spmm_blocks = (R + NC - 1) / NC;
  c->last_shape.union_spmm = 0;
  c->last_shape.fw_mfma = 0;
  c->last_tuned = 0;
  // iterations of y after every probe column had stopped (looser probe tolerance)
  c->last_y_tail = 0;
  if (B == 1 && R > 1 && prtol > rtol) {
    int probes = 0;
    for (int r = 1; r < R; ++r) probes = std::max(probes, hi[r]);
    c->last_y_tail = std::max(0, out[0].iters_y - probes);
  }
  return out;
}

}  // namespace sdgp
