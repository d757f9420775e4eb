// Jacobi-preconditioned conjugate gradients on (H + mu I) x = scale * b for the inexact
// Newton consumer, with H the BSR Hessian of ttie_eval.  Everything stays on the device: the
// scalars of the iteration are reduced from fixed-size per-block partials (fixed order, so
// the result is deterministic), every kernel re-derives them from the previous kernels'
// partials, and a convergence flag written by one kernel turns the remaining launches into
// no-ops.  Two launches per iteration:
//   k_pcg_matvec  beta = r.z(new) / r.z(old), convergence test; p' = z + beta p (formed for a
//                 row's columns as they are read, stored for the row); q = (H + mu I) p',
//                 partials of p'.q
//   k_pcg_update  alpha = r.z / p'.q; x += alpha p'; r -= alpha q; z = D^-1 r; partials r.z, r.r
// The iteration is bound by its launches and by chains of dependent loads, not by bytes (the
// matrix of a solve is a few MB and stays in the caches): eight lanes read a row's blocks side by
// side, the direction is formed where it is used instead of in a third kernel, and sums run
// through registers with one barrier.  Every sum keeps its order (a row's blocks or incidences
// one after the other; a block's rows in a fixed tree; the blocks' partials in a fixed tree), so
// the result is the same bit for bit however the work is split.  On a 1,048,576-triangle sphere
// (14,000 active rows, 150,000 blocks) an iteration's kernels took 28 us with a thread per row,
// a third kernel for the direction and sums through shared memory, now 15 us; on a cloth with springs on
// 65,536 vertices (k_pcg_hits_mf and k_pcg_rows_cp in place of k_pcg_matvec) 39 us, now
// 23 us.
//
// Active rows.  H is zero outside the rows that hold blocks (those the hits touch), so there
// (H + mu I) is mu I; with b = 0 on those rows the residual, the search direction and the
// solution stay exactly 0 on them for the whole iteration.  The solve therefore runs over the
// list of active rows only (built once per solve, in row order, so the sums keep a fixed
// order), and b must vanish elsewhere: a Newton gradient does.  On a mesh of millions of
// vertices with tens of thousands touched this makes each iteration a few microseconds.
#include "internal.h"

namespace ttie {

constexpr int kPB = 256;       // blocks of the solver's kernels; the rows of a block; threads per row kernel
constexpr int kPT = 3 * kPB;   // threads of the kernels with a thread per component
constexpr int kRowLanes = 8;
constexpr int kPR = 64 * kRowLanes;  // threads of the kernels with eight lanes per row
constexpr int kPQ = 4 * kPB;         // and their blocks

struct PcgState {
  double mu, bb, rz, rr;
  int32_t done, iters;
};

// v of the lane that the pattern names (0 where it names none)
template <int kCtrl>
__device__ __forceinline__ double dpp_of(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, 0xf, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, 0xf, 0xf, false);
  return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
// sum over the wave's lanes, in every lane (all lanes must be active): halves, quarters and so
// on added pairwise, lane l and l + 32 first
__device__ __forceinline__ double wave_total(double v) {
  v += __shfl_xor(v, 32);
  v += __shfl_xor(v, 16);
  // within a row of 16, whose halves (then quarters, ...) are equal after each step
  v += dpp_of<0x128>(v);  // row_ror 8, 4, 2, 1
  v += dpp_of<0x124>(v);
  v += dpp_of<0x122>(v);
  v += dpp_of<0x121>(v);
  return v;
}

// fixed-order sum over the kPB per-block partials of slot `slot` (every wave computes it)
__device__ __forceinline__ double grid_sum(const double* __restrict__ part, int slot) {
  const int l = __lane_id();
  const double a = part[4 * l + slot], b = part[4 * (l + 64) + slot], c = part[4 * (l + 128) + slot],
               d = part[4 * (l + 192) + slot];
  return wave_total((a + c) + (b + d));
}

// the same over partials in four parts per block, whose sum is the block's partial
__device__ __forceinline__ double grid_sum_parts(const double* __restrict__ part) {
  double v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double* w = part + 4 * (__lane_id() + 64 * k);
    v[k] = (w[0] + w[2]) + (w[1] + w[3]);
  }
  return wave_total((v[0] + v[2]) + (v[1] + v[3]));
}

// block sums of two values per row thread (threads [0, kPB)) into this block's partial slots;
// every thread of the block calls
__device__ __forceinline__ void block_partials(double v0, double v1, double* __restrict__ part) {
  __shared__ double red[2][kPB];
  if (threadIdx.x < kPB) {
    red[0][threadIdx.x] = v0;
    red[1][threadIdx.x] = v1;
  }
  __syncthreads();
  if (threadIdx.x < 128) {  // a wave per value
    const double* r = red[threadIdx.x / 64];
    const int l = threadIdx.x % 64;
    const double t = wave_total((r[l] + r[l + 128]) + (r[l + 64] + r[l + 192]));
    if (l == 0) part[4 * blockIdx.x + threadIdx.x / 64] = t;
  }
}

// diagonal block of row r (columns are sorted), or -1
__device__ __forceinline__ int64_t diag_block(const int32_t* row_ptr, const int32_t* col_idx, int64_t r) {
  int64_t lo = row_ptr[r], hi = row_ptr[r + 1] - 1;
  while (lo <= hi) {
    const int64_t mid = (lo + hi) >> 1;
    const int32_t c = col_idx[mid];
    if (c == r) return mid;
    if (c < r) lo = mid + 1; else hi = mid - 1;
  }
  return -1;
}


// ---- the active rows ------------------------------------------------------------------------
// flag[v] = row v holds blocks (row_ptr) or incidences of the last evaluation's hits; x, p = 0
// on every row, and z, p2 (the other direction vector) on an inactive one, which a column of a
// matrix whose pattern is not symmetric may name; a non-zero b there latches STATUS_INVALID.  Row n's flag is 0 (the
// scan's total).  With off, each vertex's range in the evaluation's incidence lists is written
// there too: off[v] = roff[number of touched vertices below v] for v in [0, n] (the touched
// vertices are the rows, in vertex order, and roff their list starts), so that the range of v
// is [off[v], off[v + 1]), empty when no hit touches v.
template <class S>
__global__ void __launch_bounds__(kPB) k_pcg_flags(int64_t n, const int32_t* __restrict__ row_ptr,
                                                   const uint32_t* __restrict__ bm, const uint32_t* __restrict__ wp,
                                                   const int32_t* __restrict__ roff, int32_t* __restrict__ off,
                                                   const S* __restrict__ b, S* __restrict__ x, S* __restrict__ p,
                                                   S* __restrict__ z, S* __restrict__ p2, int32_t* __restrict__ flag,
                                                   Counters* ctr) {
  for (int64_t v = (int64_t)blockIdx.x * kPB + threadIdx.x; v <= n; v += (int64_t)gridDim.x * kPB) {
    bool touched = false;
    if (off) {
      const int64_t w = v >> 5;
      const uint32_t word = bm[w], j = (uint32_t)v & 31u;
      off[v] = roff[wp[w] + (uint32_t)__popc(word & ((1u << j) - 1u))];
      touched = (word >> j) & 1u;
    }
    if (v == n) {
      flag[n] = 0;
      continue;
    }
    const bool act = (row_ptr && row_ptr[v + 1] > row_ptr[v]) || touched;
    flag[v] = act ? 1 : 0;
    bool nz = false;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[3 * v + c] = (S)0.0;
      p[3 * v + c] = (S)0.0;
      nz |= (double)b[3 * v + c] != 0.0;
    }
    if (act) continue;
#pragma unroll
    for (int c = 0; c < 3; ++c) z[3 * v + c] = p2[3 * v + c] = (S)0.0;
    if (nz) atomicCAS(&ctr->status, 0, STATUS_INVALID);
  }
}

__global__ void __launch_bounds__(kPB) k_pcg_compact(int64_t n, const int32_t* __restrict__ flag,
                                                     const int32_t* __restrict__ pos, int32_t* __restrict__ act) {
  for (int64_t v = (int64_t)blockIdx.x * kPB + threadIdx.x; v < n; v += (int64_t)gridDim.x * kPB)
    if (flag[v]) act[pos[v]] = (int32_t)v;
}

// the list of active rows and its device count (pos[n])
struct Active {
  const int32_t* rows;
  const int32_t* count;
};

template <class S>
static hipError_t pcg_active(Ctx* c, int64_t n, const int32_t* row_ptr, int32_t* off, const S* b, S* x, S* p, S* z,
                             S* p2, Active& a, hipStream_t s) {
  const Layout& L = c->L;
  int32_t* flag = wsp<int32_t>(c, L.pcg_flag);
  int32_t* pos = wsp<int32_t>(c, L.pcg_pos);
  int32_t* act = wsp<int32_t>(c, L.pcg_act);
  Counters* ctr = wsp<Counters>(c, L.counters);
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, (n + 1 + kPB - 1) / kPB));
  k_pcg_flags<S><<<g, kPB, 0, s>>>(n, row_ptr, wsp<uint32_t>(c, L.bm), wsp<uint32_t>(c, L.wp), wsp<int32_t>(c, L.roff),
                                   off, b, x, p, z, p2, flag, ctr);
  hipError_t e = launch_scan_i32(c, flag, pos, n + 1, s);
  if (e != hipSuccess) return e;
  k_pcg_compact<<<g, kPB, 0, s>>>(n, flag, pos, act);
  a.rows = act;
  a.count = pos + n;
  return hipGetLastError();
}

// a thread per active row j (blocks of kPB threads)
#define PCG_ROWS(j, a)             \
  const int64_t na_ = *(a).count; \
  for (int64_t j = (int64_t)blockIdx.x * kPB + threadIdx.x; j < na_; j += (int64_t)gridDim.x * kPB)

// A thread per component of the active rows (blocks of kPT threads): body(i, k) for row i and
// component k = 3 i + e gives the terms u v of its row's sum and u' v' of a second one; thread
// r < kPB then adds those of row r of the block's turn, component by component, to s0 and s1.
// Every block takes the same number of turns.
struct Terms {
  double u, v, u2, v2;
};
template <class Body>
__device__ __forceinline__ void pcg_components(const Active& a, double& s0, double& s1, Body body) {
  __shared__ double tu[kPT], tv[kPT], tu2[kPT], tv2[kPT];
  const int64_t na = *a.count;
  s0 = s1 = 0.0;
  for (int64_t j0 = (int64_t)blockIdx.x * kPB; j0 < na; j0 += (int64_t)gridDim.x * kPB) {
    const int64_t j = j0 + threadIdx.x / 3;
    if (j < na) {
      const int64_t i = a.rows[j];
      const Terms t = body(i, 3 * i + threadIdx.x % 3);
      tu[threadIdx.x] = t.u;
      tv[threadIdx.x] = t.v;
      tu2[threadIdx.x] = t.u2;
      tv2[threadIdx.x] = t.v2;
    }
    __syncthreads();
    if (threadIdx.x < kPB && j0 + threadIdx.x < na) {
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const int k = 3 * threadIdx.x + e;
        s0 += tu[k] * tv[k];
        s1 += tu2[k] * tv2[k];
      }
    }
    __syncthreads();
  }
}

// Eight lanes per active row: body(i, sub, lds) gives, in lanes sub < 3, the terms of component
// sub, summed like those of pcg_components.  lds: the wave's 64 x 3 doubles.  The 256 rows of
// a block of the row kernels go to four blocks here (a few thousand active rows then reach
// every CU): part m takes the rows m, m + 4, ... of each quarter of 64, which is where the fixed tree
// over the 256 splits, and leaves its sum in part[4 b + m].
template <class Body>
__device__ __forceinline__ void pcg_rows(const Active& a, double* __restrict__ part, Body body) {
  __shared__ double tu[64][3], tv[64][3], lds[kPR][3];
  const int64_t na = *a.count;
  const int sub = threadIdx.x % kRowLanes, u = threadIdx.x / kRowLanes;
  // (the four parts of a block's rows on one XCD, every eighth block: they share cache lines)
  const int64_t b = blockIdx.x / 32 * 8 + blockIdx.x % 8;
  const int m = blockIdx.x / 8 % 4;
  const auto row_of = [m](int v) { return m + 4 * (v & 15) + 64 * (v >> 4); };
  double s0 = 0.0;
  for (int64_t j0 = b * kPB; j0 < na; j0 += (int64_t)kPB * kPB) {
    if (j0 + row_of(u) < na) {
      const Terms t = body((int64_t)a.rows[j0 + row_of(u)], sub, lds + (threadIdx.x & ~63u));
      if (sub < 3) {
        tu[u][sub] = t.u;
        tv[u][sub] = t.v;
      }
    }
    __syncthreads();
    if (threadIdx.x < 64 && j0 + row_of(threadIdx.x) < na) {
#pragma unroll
      for (int e = 0; e < 3; ++e) s0 += tu[threadIdx.x][e] * tv[threadIdx.x][e];
    }
    __syncthreads();
  }
  if (threadIdx.x < 64) {
    s0 = wave_total(s0);
    if (threadIdx.x == 0) part[4 * b + m] = s0;
  }
}

// Adds the three-component terms term(k, t) of k in [beg, end) to acc, one after the other:
// eight lanes form eight terms at a time, and lane e < 3 of them adds the components e (its acc
// is the result).
template <class Term>
__device__ __forceinline__ double ordered_sum(int32_t beg, int32_t end, int sub, double (*lds)[3], double acc, Term term) {
  const int lane = __lane_id(), first = lane & ~(kRowLanes - 1);
  for (int32_t k0 = beg; k0 < end; k0 += kRowLanes) {
    if (k0 + sub < end) {
      double t[3];
      term(k0 + sub, t);
#pragma unroll
      for (int e = 0; e < 3; ++e) lds[lane][e] = t[e];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (sub < 3) {
      const int n = min(kRowLanes, end - k0);
      double t[kRowLanes];
#pragma unroll
      for (int s = 0; s < kRowLanes; ++s) t[s] = lds[first + s][sub];  // (past n: not added)
#pragma unroll
      for (int s = 0; s < kRowLanes; ++s)
        if (s < n) acc += t[s];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  return acc;
}

// The start of an iteration, every wave alike: beta and the convergence test of the iteration
// before it (rz_new NULL: there is none, beta = 0).  False when the solve is over.
__device__ __forceinline__ bool next_direction(const double* __restrict__ rz_old, const double* __restrict__ rz_new,
                                               const double* __restrict__ setup_part, double tol, int iter,
                                               PcgState* st, double& beta) {
  beta = 0.0;
  if (st->done) return false;
  if (!rz_new) return true;
  const double rzo = grid_sum(rz_old, 0), rzn = grid_sum(rz_new, 0), rr = grid_sum(rz_new, 1),
               bb = grid_sum(setup_part, 1);
  const bool conv = rr <= tol * tol * bb;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->iters = iter;
    st->rr = rr;
    st->bb = bb;
    if (conv) st->done = 1;
  }
  if (rzo > 0.0) beta = rzn / rzo;
  return !conv;
}
// p' = z + beta p at component k, rounded to the vectors' type
template <class S>
__device__ __forceinline__ double direction(const S* __restrict__ z, const S* __restrict__ p, double beta, int64_t k) {
  return (double)(S)((double)z[k] + beta * (double)p[k]);
}

template <class S>
__global__ void __launch_bounds__(kPB) k_pcg_diag(Active a, const int32_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ col_idx, const S* __restrict__ vals,
                                                  double* __restrict__ part) {
  double sum = 0.0, cnt = 0.0;
  PCG_ROWS(j, a) {
    const int64_t r = a.rows[j];
    const int64_t d = diag_block(row_ptr, col_idx, r);
    if (d >= 0) {
      sum += (double)vals[9 * d] + (double)vals[9 * d + 4] + (double)vals[9 * d + 8];
      cnt += 3.0;
    }
  }
  block_partials(sum, cnt, part);
}

template <class S>
__global__ void __launch_bounds__(kPB) k_pcg_setup(Active a, const int32_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col_idx, const S* __restrict__ vals,
                                                   const S* __restrict__ b, double scale, S* __restrict__ r,
                                                   S* __restrict__ z, S* __restrict__ p, S* __restrict__ dinv,
                                                   double mu_rel, const double* __restrict__ pdiag,
                                                   double* __restrict__ pout, PcgState* st) {
  const double dsum = grid_sum(pdiag, 0), dcnt = grid_sum(pdiag, 1);
  // mu relative to the mean diagonal entry of the rows holding blocks (1 for an empty matrix)
  const double mu = mu_rel * (dcnt > 0.0 ? dsum / dcnt : 1.0);
  double rz = 0.0, bb = 0.0;
  PCG_ROWS(j, a) {
    const int64_t i = a.rows[j];
    const int64_t d = diag_block(row_ptr, col_idx, i);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double dg = (d >= 0 ? (double)vals[9 * d + 4 * c] : 0.0) + mu;
      const double di = dg > 0.0 ? 1.0 / dg : 1.0;
      const double ri = scale * (double)b[3 * i + c];
      const double zi = di * ri;
      dinv[3 * i + c] = (S)di;
      r[3 * i + c] = (S)ri;
      z[3 * i + c] = (S)zi;
      p[3 * i + c] = (S)zi;
      rz += ri * zi;
      bb += ri * ri;
    }
  }
  block_partials(rz, bb, pout);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->mu = mu;
    st->bb = st->rr = 0.0;
    st->done = 0;
    st->iters = 0;
  }
}

// row i of a BSR matrix times the vector whose component k is vec(k), added to acc (ordered_sum)
template <class S, class Vec>
__device__ __forceinline__ double row_product(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                              const S* __restrict__ vals, Vec vec, int64_t i, int sub, double (*lds)[3],
                                              double acc) {
  return ordered_sum(row_ptr[i], row_ptr[i + 1], sub, lds, acc, [=](int32_t k, double (&t)[3]) {
    const int64_t c = 3 * (int64_t)col_idx[k];
    const double p0 = vec(c), p1 = vec(c + 1), p2 = vec(c + 2);
    const S* v = vals + 9 * (int64_t)k;
#pragma unroll
    for (int e = 0; e < 3; ++e) t[e] = (double)v[3 * e] * p0 + (double)v[3 * e + 1] * p1 + (double)v[3 * e + 2] * p2;
  });
}

template <class S>
__global__ void __launch_bounds__(kPR) k_pcg_matvec(Active a, const int32_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col_idx, const S* __restrict__ vals,
                                                    const S* __restrict__ z, const S* __restrict__ p,
                                                    S* __restrict__ pn, S* __restrict__ q,
                                                    double* __restrict__ pq_part, const double* __restrict__ rz_old,
                                                    const double* __restrict__ rz_new,
                                                    const double* __restrict__ setup_part, double tol, int iter,
                                                    PcgState* st) {
  double beta;
  if (!next_direction(rz_old, rz_new, setup_part, tol, iter, st, beta)) return;
  const double mu = st->mu;
  pcg_rows(a, pq_part, [&](int64_t i, int sub, double (*lds)[3]) {
    const int64_t k = 3 * i + min(sub, 2);
    const double pi = direction(z, p, beta, k);
    const double qi = row_product(row_ptr, col_idx, vals, [=](int64_t c) { return direction(z, p, beta, c); }, i, sub,
                                  lds, mu * pi);
    if (sub < 3) {
      pn[k] = (S)pi;
      q[k] = (S)qi;
    }
    return Terms{pi, qi, 0.0, 0.0};
  });
}

template <class S>
__global__ void __launch_bounds__(kPT) k_pcg_update(Active a, S* __restrict__ x, S* __restrict__ r,
                                                    S* __restrict__ z, const S* __restrict__ p,
                                                    const S* __restrict__ q, const S* __restrict__ dinv,
                                                    const double* __restrict__ rz_part, const double* __restrict__ pq_part,
                                                    double* __restrict__ out_part, PcgState* st) {
  if (st->done) return;
  const double rz = grid_sum(rz_part, 0), pq = grid_sum_parts(pq_part);
  if (!(pq > 0.0)) {  // (H + mu I) should be positive definite; stop on a breakdown
    if (blockIdx.x == 0 && threadIdx.x == 0) st->done = 2;
    return;
  }
  const double alpha = rz / pq;
  double rzn, rr;
  pcg_components(a, rzn, rr, [&](int64_t, int64_t k) {
    x[k] = (S)((double)x[k] + alpha * (double)p[k]);
    const double ri = (double)r[k] - alpha * (double)q[k];
    const double zi = (double)dinv[k] * ri;
    r[k] = (S)ri;
    z[k] = (S)zi;
    return Terms{ri, zi, ri, ri};
  });
  block_partials(rzn, rr, out_part);
}

// ---- matrix-free variant: H applied from the last evaluation's per-hit records -------------
// H = sum over hits of J^T M J with J = [a^T; b^T] (2 x 18), the PSD core M of the
// evaluation.  Rows gather their incidences in pair-key order (the sorted lists the
// evaluation leaves behind), so the products are deterministic.

// Per iteration one launch more than with the matrix: k_pcg_hits_mf forms the direction (for
// the active rows, and where the hits read it) and the hits' products, k_pcg_rows_mf gathers
// them.

// raw diagonal of H per dof into dg, partials of (sum, count) over the active rows, as the BSR
// variant takes them over the rows holding blocks
template <class S>
__global__ void __launch_bounds__(kPB) k_pcg_diag_mf(Active a, const int32_t* __restrict__ off,
                                                     const Incidence* __restrict__ inc,
                                                     const AsmRec<S>* __restrict__ recs, S* __restrict__ dg,
                                                     double* __restrict__ part) {
  double sum = 0.0, cnt = 0.0;
  PCG_ROWS(j, a) {
    const int64_t i = a.rows[j];
    const int32_t b = off[i], e = off[i + 1];
    double d[3] = {0.0, 0.0, 0.0};
    for (int32_t k = b; k < e; ++k) {
      const Incidence in = inc[k];
      const AsmRec<S>& r = recs[in.hit];
      const int s = in.slot;
      for (int l = 0; l < 6; ++l) {
        if (r.vid[l] != r.vid[s]) continue;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double as = r.a[3 * s + c], bs = r.b[3 * s + c], al = r.a[3 * l + c], bl = r.b[3 * l + c];
          d[c] += (double)r.M[0] * as * al + (double)r.M[1] * (as * bl + bs * al) + (double)r.M[2] * bs * bl;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) dg[3 * i + c] = (S)d[c];
    if (e > b) {
      sum += d[0] + d[1] + d[2];
      cnt += 3.0;
    }
  }
  block_partials(sum, cnt, part);
}

// as k_pcg_setup, with the diagonal from dinv (holding the raw diagonal on entry)
template <class S>
__global__ void __launch_bounds__(kPB) k_pcg_setup_mf(Active a, const S* __restrict__ b, double scale,
                                                      S* __restrict__ r, S* __restrict__ z, S* __restrict__ p,
                                                      S* __restrict__ dinv, double mu_rel,
                                                      const double* __restrict__ pdiag, double* __restrict__ pout,
                                                      PcgState* st) {
  const double dsum = grid_sum(pdiag, 0), dcnt = grid_sum(pdiag, 1);
  const double mu = mu_rel * (dcnt > 0.0 ? dsum / dcnt : 1.0);
  double rz = 0.0, bb = 0.0;
  PCG_ROWS(j, a) {
    const int64_t i = a.rows[j];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int64_t k = 3 * i + c;
      const double dg = (double)dinv[k] + mu;
      const double di = dg > 0.0 ? 1.0 / dg : 1.0;
      const double ri = scale * (double)b[k];
      const double zi = di * ri;
      dinv[k] = (S)di;
      r[k] = (S)ri;
      z[k] = (S)zi;
      p[k] = (S)zi;
      rz += ri * zi;
      bb += ri * ri;
    }
  }
  block_partials(rz, bb, pout);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->mu = mu;
    st->bb = st->rr = 0.0;
    st->done = 0;
    st->iters = 0;
  }
}

// the direction p' on the active rows, and per hit hv = J^T M (J p'_local), 18 values.  Eight
// lanes per hit, lane s < 6 with slot s: each adds its three terms to the sums of the lane
// before it, so a hit's 18 terms are added in slot order.
constexpr int kHitLanes = 8;

template <class S>
__global__ void __launch_bounds__(kPT) k_pcg_hits_mf(Active a, const AsmRec<S>* __restrict__ recs, const Counters* ctr,
                                                     uint32_t max_hits, const S* __restrict__ z,
                                                     const S* __restrict__ p, S* __restrict__ pn, S* __restrict__ hv,
                                                     const double* __restrict__ rz_old,
                                                     const double* __restrict__ rz_new,
                                                     const double* __restrict__ setup_part, double tol, int iter,
                                                     PcgState* st) {
  double beta;
  if (!next_direction(rz_old, rz_new, setup_part, tol, iter, st, beta)) return;
  const uint32_t H = min(ctr->last_hits, max_hits);
  const int sub = threadIdx.x % kHitLanes;
  for (uint32_t h = (blockIdx.x * kPT + threadIdx.x) / kHitLanes; h < H; h += gridDim.x * kPT / kHitLanes) {
    const AsmRec<S>& r = recs[h];
    double av[3] = {0.0, 0.0, 0.0}, bv[3] = {0.0, 0.0, 0.0}, pv[3] = {0.0, 0.0, 0.0};
    if (sub < 6) {
      const int64_t k = 3 * (int64_t)r.vid[sub];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        pv[c] = direction(z, p, beta, k + c);
        av[c] = (double)r.a[3 * sub + c];
        bv[c] = (double)r.b[3 * sub + c];
      }
    }
    double ua = 0.0, ub = 0.0;
#pragma unroll
    for (int s = 0; s < 6; ++s) {
      // (in turn s only lane s's sums matter: lane s - 1 made its own in the turn before)
      ua = s ? dpp_of<0x111>(ua) : 0.0;
      ub = s ? dpp_of<0x111>(ub) : 0.0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ua += av[c] * pv[c];
        ub += bv[c] * pv[c];
      }
    }
    const int last = (__lane_id() & ~(kHitLanes - 1)) + 5;
    ua = __shfl(ua, last);
    ub = __shfl(ub, last);
    const double wa = (double)r.M[0] * ua + (double)r.M[1] * ub, wb = (double)r.M[1] * ua + (double)r.M[2] * ub;
    if (sub < 6) {
#pragma unroll
      for (int c = 0; c < 3; ++c) hv[18 * (int64_t)h + 3 * sub + c] = (S)(wa * av[c] + wb * bv[c]);
    }
  }
  const int64_t nd = 3 * (int64_t)*a.count;
  for (int64_t t = (int64_t)blockIdx.x * kPT + threadIdx.x; t < nd; t += (int64_t)gridDim.x * kPT) {
    const int64_t k = 3 * (int64_t)a.rows[t / 3] + t % 3;
    pn[k] = (S)direction(z, p, beta, k);
  }
}

// the hit products of row i's incidences, in their order, added to acc (ordered_sum)
template <class S>
__device__ __forceinline__ double gather_hits(const int32_t* __restrict__ off, const Incidence* __restrict__ inc,
                                              const S* __restrict__ hv, int64_t i, int sub, double (*lds)[3], double acc) {
  return ordered_sum(off[i], off[i + 1], sub, lds, acc, [=](int32_t k, double (&t)[3]) {
    const Incidence in = inc[k];
#pragma unroll
    for (int e = 0; e < 3; ++e) t[e] = (double)hv[18 * (int64_t)in.hit + 3 * in.slot + e];
  });
}

// q = (H + mu I) p from the per-hit products; partials of p.q
template <class S>
__global__ void __launch_bounds__(kPR) k_pcg_rows_mf(Active a, const int32_t* __restrict__ off,
                                                     const Incidence* __restrict__ inc, const S* __restrict__ hv,
                                                     const S* __restrict__ p, S* __restrict__ q,
                                                     double* __restrict__ pq_part, const PcgState* st) {
  if (st->done) return;
  const double mu = st->mu;
  pcg_rows(a, pq_part, [&](int64_t i, int sub, double (*lds)[3]) {
    const int64_t k = 3 * i + min(sub, 2);
    const double pi = p[k], qi = gather_hits(off, inc, hv, i, sub, lds, mu * pi);
    if (sub < 3) q[k] = (S)qi;
    return Terms{pi, qi, 0.0, 0.0};
  });
}

// ---- coupled variant: A = K + w H + mu I, K a caller's PSD BSR matrix (FP64) --------------
// (the quasi-static objective's elastic Hessian), H applied from the hit records as above.
// Jacobi diagonal: K's diagonal entries + w times H's + mu.
__global__ void __launch_bounds__(kPB) k_pcg_setup_cp(Active a, const int32_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ col_idx,
                                                      const double* __restrict__ vals, double w, double mu,
                                                      const double* __restrict__ b, double scale,
                                                      double* __restrict__ r, double* __restrict__ z,
                                                      double* __restrict__ p, double* __restrict__ dinv,
                                                      double* __restrict__ pout, PcgState* st) {
  double rz = 0.0, bb = 0.0;
  PCG_ROWS(j, a) {
    const int64_t i = a.rows[j];
    const int64_t d = diag_block(row_ptr, col_idx, i);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double dg = (d >= 0 ? vals[9 * d + 4 * c] : 0.0) + w * dinv[3 * i + c] + mu;
      const double di = dg > 0.0 ? 1.0 / dg : 1.0;
      const double ri = scale * b[3 * i + c];
      const double zi = di * ri;
      dinv[3 * i + c] = di;
      r[3 * i + c] = ri;
      z[3 * i + c] = zi;
      p[3 * i + c] = zi;
      rz += ri * zi;
      bb += ri * ri;
    }
  }
  block_partials(rz, bb, pout);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->mu = mu;
    st->bb = st->rr = 0.0;
    st->done = 0;
    st->iters = 0;
  }
}

// q = (K + w H + mu I) p: K's row times p, plus w times the gathered hit products; partials of p.q
__global__ void __launch_bounds__(kPR) k_pcg_rows_cp(Active a, const int32_t* __restrict__ off,
                                                     const Incidence* __restrict__ inc, const double* __restrict__ hv,
                                                     const int32_t* __restrict__ row_ptr,
                                                     const int32_t* __restrict__ col_idx,
                                                     const double* __restrict__ vals, double w,
                                                     const double* __restrict__ p, double* __restrict__ q,
                                                     double* __restrict__ pq_part, const PcgState* st) {
  if (st->done) return;
  const double mu = st->mu;
  pcg_rows(a, pq_part, [&](int64_t i, int sub, double (*lds)[3]) {
    const int64_t k = 3 * i + min(sub, 2);
    const double pi = p[k], hs = gather_hits(off, inc, hv, i, sub, lds, 0.0);
    const double qi =
        row_product(row_ptr, col_idx, vals, [=](int64_t c) { return p[c]; }, i, sub, lds, mu * pi + w * hs);
    if (sub < 3) q[k] = qi;
    return Terms{pi, qi, 0.0, 0.0};
  });
}

template <class S>
__global__ void __launch_bounds__(kPB) k_pcg_xb(Active a, const S* __restrict__ x, const S* __restrict__ b,
                                                double scale, double* __restrict__ part) {
  double xb = 0.0;
  PCG_ROWS(j, a) {
    const int64_t i = a.rows[j];
#pragma unroll
    for (int c = 0; c < 3; ++c) xb += (double)x[3 * i + c] * scale * (double)b[3 * i + c];
  }
  block_partials(xb, 0.0, part);
}

// rz_last: the partials of the last iteration's residual (NULL without iterations), whose test
// no later iteration has made
__global__ void __launch_bounds__(64) k_pcg_info(const double* __restrict__ part, const double* __restrict__ rz_last,
                                                 const double* __restrict__ setup_part, int max_iter,
                                                 const PcgState* st, double* info) {
  const double xb = grid_sum(part, 0);
  double rr = st->rr, bb = st->bb;
  int32_t iters = st->iters;
  if (rz_last && !st->done) {
    rr = grid_sum(rz_last, 1);
    bb = grid_sum(setup_part, 1);
    iters = max_iter;
  }
  if (threadIdx.x == 0) {
    info[0] = iters;
    info[1] = bb > 0.0 ? sqrt(rr / bb) : 0.0;
    info[2] = st->mu;
    info[3] = xb;
  }
}

template <class S>
__global__ void __launch_bounds__(kPB) k_axpy(int64_t n, double alpha, const double* __restrict__ x,
                                              const S* __restrict__ d, double* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * kPB + threadIdx.x; i < n; i += (int64_t)gridDim.x * kPB) {
    const double v = x[i] + alpha * (double)d[i];
    out[i] = fabs(v) < 0x1p-200 ? 0.0 : v;  // stay in the predicates' coordinate domain
  }
}


// the vectors and partials of a solve, carved from the workspace
template <class S>
struct PcgBufs {
  S *r, *z, *p[2], *q, *dinv;  // p: the direction of the iterations in turn
  double *pdiag, *pset, *pq, *prz[2];
  PcgState* st;
  PcgBufs(Ctx* c) {
    const Layout& L = c->L;
    S* base = wsp<S>(c, L.pcg_vec);
    const int64_t m3 = 3 * (int64_t)c->lim.max_verts;
    r = base;
    z = base + m3;
    p[0] = base + 2 * m3;
    q = base + 3 * m3;
    dinv = base + 4 * m3;
    p[1] = base + 5 * m3;
    double* part = wsp<double>(c, L.pcg_part);  // 5 partial arrays of kPB x 4
    pdiag = part;
    pset = part + 4 * kPB;
    pq = part + 8 * kPB;
    prz[0] = part + 12 * kPB;
    prz[1] = part + 16 * kPB;
    st = wsp<PcgState>(c, L.pcg_state);
  }
  // the partials of r.z, r.r that iteration it starts from (before iteration 0: the setup's)
  // and those of the iteration before
  double* rz_of(int it) const { return it == 0 ? pset : prz[(it - 1) % 2]; }
};

// The iterations of a solve: product(it, rz_old, rz_new) launches the kernels that form the
// direction and its product, k_pcg_update the rest; then the caller's four numbers.
template <class S, class Product>
static void pcg_iterate(const Active& a, const PcgBufs<S>& B, const S* b, double scale, S* x, int max_iter, double* info,
                        hipStream_t s, Product product) {
  for (int it = 0; it < max_iter; ++it) {
    product(it, it ? B.rz_of(it - 1) : nullptr, it ? B.rz_of(it) : nullptr);
    k_pcg_update<S><<<kPB, kPT, 0, s>>>(a, x, B.r, B.z, B.p[(it + 1) % 2], B.q, B.dinv, B.rz_of(it), B.pq,
                                        B.rz_of(it + 1), B.st);
  }
  if (info) {
    k_pcg_xb<S><<<kPB, kPB, 0, s>>>(a, x, b, scale, B.pq);
    k_pcg_info<<<1, 64, 0, s>>>(B.pq, max_iter ? B.rz_of(max_iter) : nullptr, B.pset, max_iter, B.st, info);
  }
}

template <class S>
static hipError_t pcg_impl(Ctx* c, int64_t n, const int32_t* row_ptr, const int32_t* col_idx, const S* vals,
                           const S* b, double scale, S* x, double mu_rel, int max_iter, double tol, double* info,
                           hipStream_t s) {
  PcgBufs<S> B(c);
  stage_begin(c, TTIE_STAGE_PCG, s);
  Active a;
  hipError_t e = pcg_active<S>(c, n, row_ptr, nullptr, b, x, B.p[0], B.z, B.p[1], a, s);
  if (e != hipSuccess) return e;
  k_pcg_diag<S><<<kPB, kPB, 0, s>>>(a, row_ptr, col_idx, vals, B.pdiag);
  k_pcg_setup<S><<<kPB, kPB, 0, s>>>(a, row_ptr, col_idx, vals, b, scale, B.r, B.z, B.p[0], B.dinv, mu_rel, B.pdiag,
                                     B.pset, B.st);
  pcg_iterate<S>(a, B, b, scale, x, max_iter, info, s, [&](int it, const double* rz_old, const double* rz_new) {
    k_pcg_matvec<S><<<kPQ, kPR, 0, s>>>(a, row_ptr, col_idx, vals, B.z, B.p[it % 2], B.p[(it + 1) % 2], B.q, B.pq, rz_old,
                                        rz_new, B.pset, tol, it, B.st);
  });
  stage_end(c, TTIE_STAGE_PCG, s);
  return hipGetLastError();
}

template <class S>
static hipError_t pcg_mf_impl(Ctx* c, int64_t n, const S* b, double scale, S* x, double mu_rel, int max_iter, double tol,
                              double* info, hipStream_t s) {
  const Layout& L = c->L;
  PcgBufs<S> B(c);
  const AsmRec<S>* recs = wsp<AsmRec<S>>(c, L.recs);
  int32_t* off = wsp<int32_t>(c, L.off);
  const Incidence* inc = wsp<Incidence>(c, L.inc2);
  S* hv = wsp<S>(c, L.hvbuf);
  const Counters* ctr = wsp<Counters>(c, L.counters);
  const uint32_t max_hits = (uint32_t)c->lim.max_hits;
  stage_begin(c, TTIE_STAGE_PCG, s);
  Active a;
  hipError_t e = pcg_active<S>(c, n, nullptr, off, b, x, B.p[0], B.z, B.p[1], a, s);
  if (e != hipSuccess) return e;
  k_pcg_diag_mf<S><<<kPB, kPB, 0, s>>>(a, off, inc, recs, B.dinv, B.pdiag);
  k_pcg_setup_mf<S><<<kPB, kPB, 0, s>>>(a, b, scale, B.r, B.z, B.p[0], B.dinv, mu_rel, B.pdiag, B.pset, B.st);
  pcg_iterate<S>(a, B, b, scale, x, max_iter, info, s, [&](int it, const double* rz_old, const double* rz_new) {
    k_pcg_hits_mf<S><<<kPB, kPT, 0, s>>>(a, recs, ctr, max_hits, B.z, B.p[it % 2], B.p[(it + 1) % 2], hv, rz_old, rz_new,
                                         B.pset, tol, it, B.st);
    k_pcg_rows_mf<S><<<kPQ, kPR, 0, s>>>(a, off, inc, hv, B.p[(it + 1) % 2], B.q, B.pq, B.st);
  });
  stage_end(c, TTIE_STAGE_PCG, s);
  return hipGetLastError();
}

hipError_t launch_pcg_coupled(Ctx* c, int64_t n, const int32_t* row_ptr, const int32_t* col_idx, const double* vals,
                              double w, const double* b, double scale, double* x, double mu, int max_iter, double tol,
                              double* info, hipStream_t s) {
  const Layout& L = c->L;
  PcgBufs<double> B(c);
  const AsmRec<double>* recs = wsp<AsmRec<double>>(c, L.recs);
  int32_t* off = wsp<int32_t>(c, L.off);
  const Incidence* inc = wsp<Incidence>(c, L.inc2);
  double* hv = wsp<double>(c, L.hvbuf);
  const Counters* ctr = wsp<Counters>(c, L.counters);
  const uint32_t max_hits = (uint32_t)c->lim.max_hits;
  stage_begin(c, TTIE_STAGE_PCG, s);
  Active a;
  hipError_t e = pcg_active<double>(c, n, row_ptr, off, b, x, B.p[0], B.z, B.p[1], a, s);
  if (e != hipSuccess) return e;
  k_pcg_diag_mf<double><<<kPB, kPB, 0, s>>>(a, off, inc, recs, B.dinv, B.pdiag);  // raw diagonal of H into dinv
  k_pcg_setup_cp<<<kPB, kPB, 0, s>>>(a, row_ptr, col_idx, vals, w, mu, b, scale, B.r, B.z, B.p[0], B.dinv, B.pset,
                                     B.st);
  pcg_iterate<double>(a, B, b, scale, x, max_iter, info, s, [&](int it, const double* rz_old, const double* rz_new) {
    k_pcg_hits_mf<double><<<kPB, kPT, 0, s>>>(a, recs, ctr, max_hits, B.z, B.p[it % 2], B.p[(it + 1) % 2], hv, rz_old,
                                              rz_new, B.pset, tol, it, B.st);
    k_pcg_rows_cp<<<kPQ, kPR, 0, s>>>(a, off, inc, hv, row_ptr, col_idx, vals, w, B.p[(it + 1) % 2], B.q, B.pq, B.st);
  });
  stage_end(c, TTIE_STAGE_PCG, s);
  return hipGetLastError();
}

hipError_t launch_pcg_mf(Ctx* c, int64_t n, const void* b, double scale, void* x, double mu_rel, int max_iter,
                         double tol, double* info, hipStream_t s) {
  if (c->last_precision == TTIE_FP64)
    return pcg_mf_impl<double>(c, n, (const double*)b, scale, (double*)x, mu_rel, max_iter, tol, info, s);
  return pcg_mf_impl<float>(c, n, (const float*)b, scale, (float*)x, mu_rel, max_iter, tol, info, s);
}

hipError_t launch_pcg(Ctx* c, int64_t n, const int32_t* row_ptr, const int32_t* col_idx, const void* vals,
                      const void* b, double scale, void* x, double mu_rel, int max_iter, double tol, int precision,
                      double* info, hipStream_t s) {
  if (precision == TTIE_FP64)
    return pcg_impl<double>(c, n, row_ptr, col_idx, (const double*)vals, (const double*)b, scale, (double*)x, mu_rel,
                            max_iter, tol, info, s);
  return pcg_impl<float>(c, n, row_ptr, col_idx, (const float*)vals, (const float*)b, scale, (float*)x, mu_rel,
                         max_iter, tol, info, s);
}

hipError_t launch_axpy(int64_t n_verts, double alpha, const double* x, const void* d, double* out, int precision,
                       hipStream_t s) {
  const int64_t n = 3 * n_verts;
  const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, (n + kPB - 1) / kPB));
  if (precision == TTIE_FP64)
    k_axpy<double><<<g, kPB, 0, s>>>(n, alpha, x, (const double*)d, out);
  else
    k_axpy<float><<<g, kPB, 0, s>>>(n, alpha, x, (const float*)d, out);
  return hipGetLastError();
}

}  // namespace ttie
