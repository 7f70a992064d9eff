// gfx950 inverses by blocked LU elimination with partial pivoting: the
// coarsest operator (banded under the ordering chosen at setup) and the dense
// Schwarz blocks.
//
// Two launches.  k_lu factors each matrix in one workgroup, panel by panel of
// 16 columns.  Pivots are searched only among the rows that still wait for
// one, by a single wave that holds them in registers, so a pivot step needs no
// workgroup barrier; the other waves meanwhile apply the previous panel to
// the columns beyond the current one on the matrix cores.  k_lu_rows then
// finds rows of the inverse, 16 G at a time, from the factors: these
// workgroups are independent and fill the device.
//
// Factors, in place: rows are never exchanged, perm[s] is the pivot row of
// step s.  With R_p the 16 pivot rows of panel p, B_p their entries in the
// panel's columns, the panel's columns hold B_p^-1 on the rows R_p (row of
// step s: row s of B_p^-1, its columns in step order) and PC = -A B_p^-1 on
// the rows still waiting, which are updated by
//     A[i][j] += sum_t PC[i][t] A[perm[16 p + t]][j]
// for the columns j beyond the panel; a pivot row keeps its values there.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <climits>
#include <mutex>

#include "fsi_kernels.h"
#include "fsi_pivot.h"

namespace fsi {

constexpr int kLuNb = 16;                        // panel width: one matrix-core tile
constexpr int kLuThreads = 512, kLuWaves = kLuThreads / 64;
constexpr int kLuAhead = 4;                      // C tiles in flight per wave in the updates
// stride of a panel row in LDS: 16-byte aligned, and the 16 rows of a tile
// start 4 banks apart, so the 16-byte operand reads do not conflict
template <typename T>
constexpr int kLuStride = sizeof(T) == 8 ? 18 : 20;

// four consecutive elements (the operand of one lane of a 16x16 panel tile)
template <typename T>
struct alignas(16) Quad {
  T v[4];
};

// the pivot row (lane ll, register row ql) into scalars
template <typename T, int R, int Q = 0>
__device__ __forceinline__ void lu_take(const T (&v)[R][kLuNb], int ql, int ll, T (&prow)[kLuNb]) {
  if (Q == R - 1 || ql == Q) {
#pragma unroll
    for (int c = 0; c < kLuNb; ++c) prow[c] = readlane(v[Q][c], ll);
  } else if constexpr (Q + 1 < R) {
    lu_take<T, R, Q + 1>(v, ql, ll, prow);
  }
}

// One panel of 16 columns factored by one wave.  Lane l holds the rows of
// slots l + 64 q in v[q]; step[q] is -1 for a row that waits for its pivot (a
// candidate), and becomes the step at which it is the pivot; other slots hold
// zeros and a step >= 16.  Every row is eliminated in every column of the panel
// (Gauss-Jordan inside the panel), so that the rows end as described above; a
// pivot row stays unscaled until the end (1 in its own column, and it takes
// the later eliminations like any other), so that a step has no branch that
// moves rows between registers.  Returns 0, or 1 + the first step (0-based, in
// the panel) whose pivot is zero or not finite (the steps go on without a
// branch; the result is unusable).
template <typename T, int R>
__device__ __forceinline__ int lu_panel(T (&v)[R][kLuNb], int (&step)[R]) {
  const int lane = threadIdx.x & 63;
  int fail = 0;
  T scale[R];
#pragma unroll
  for (int q = 0; q < R; ++q) scale[q] = 1;
#pragma unroll
  for (int t = 0; t < kLuNb; ++t) {
    double key = -1.0;
    T sv = 1;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const double kq = pivot_key((double)v[q][t], q * 64 + lane);
      if (step[q] < 0 && kq > key) {
        key = kq;
        sv = v[q][t];
      }
    }
    const T dl = recip(sv);   // every lane inverts its own candidate during the reduction
    const double best = wave_max<true>(key);
    const double bv = key_value(best);
    const bool bad = !(best >= 0.0) || !(bv > 0.0) || bv >= key_value(pivot_key(DBL_MAX, 0));
    fail = fail == 0 && bad ? t + 1 : fail;
    const int slot = __builtin_amdgcn_readfirstlane(key_row(best));
    const int ll = slot & 63;
    const T d = readlane(dl, ll);
    T prow[kLuNb];
    lu_take<T, R>(v, slot >> 6, ll, prow);
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const bool own = slot == q * 64 + lane;
      const T fd = own ? (T)0 : v[q][t] * d;
      scale[q] = own ? d : scale[q];
      step[q] = own ? t : step[q];
#pragma unroll
      for (int c = 0; c < kLuNb; ++c) v[q][c] = c == t ? (own ? (T)1 : -fd) : v[q][c] - fd * prow[c];
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q)
#pragma unroll
    for (int c = 0; c < kLuNb; ++c) v[q][c] *= scale[q];
  return fail;
}

// Shared memory of a factorization, by the parity of a panel: its rows (first
// the panel being factored, then its factors for the updates), the matrix row
// in each slot or -1, the panel's pivot rows in step order, the slots in use
// or the failure; and (banded) the panel at which each slot's row entered.
template <typename T>
struct LuLds {
  T *base;
  int *ints;
  int nslot;
  __device__ __forceinline__ T *panel(int p) const { return base + (p & 1) * nslot * kLuStride<T>; }
  __device__ __forceinline__ int *row(int p) const { return ints + (p & 1) * nslot; }
  __device__ __forceinline__ int *entry() const { return ints + 2 * nslot; }
  __device__ __forceinline__ int *piv(int p) const { return ints + 3 * nslot + (p & 1) * kLuNb; }
  __device__ __forceinline__ int *result(int p) const { return ints + 3 * nslot + 2 * kLuNb + (p & 1); }
};
static inline size_t lu_lds_bytes(int nslot, size_t elem, int stride) {
  return 2 * (size_t)nslot * stride * elem + sizeof(int) * (3 * (size_t)nslot + 2 * kLuNb + 4);
}

// The factoring wave's part of panel p: the rows of slots [0, cnt) from LDS
// (with the panel's columns up to date), their factors to LDS and to the
// matrix, and the slots of the next panel.  Banded: a row keeps its slot
// until it is a pivot, freed slots go to the rows [hi, hinext) that enter
// next.  Dense: the rows left are moved together.  Returns the slots in use
// for the next panel, or -1 - step on a failing pivot.
template <typename T, int R, bool BAND>
__device__ __forceinline__ int lu_factor(T *__restrict__ A, int64_t ld, int p, int w, int cnt, int hi,
                                         int hinext, const LuLds<T> &L, int *__restrict__ perm,
                                         int *__restrict__ plo) {
  constexpr int LS = kLuStride<T>;
  const int lane = threadIdx.x & 63, p0 = p * kLuNb;
  const unsigned long long below = (1ull << lane) - 1;
  T *P = L.panel(p);
  const int *row = L.row(p);
  int *rown = L.row(p + 1);
  T v[R][kLuNb];
  int ri[R], step[R];
  int unit = kLuNb - w;   // a last panel of w < 16 columns: the other pivots are unit rows in free slots
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int s = q * 64 + lane;
    ri[q] = s < cnt ? row[s] : -1;
    const unsigned long long fr = __ballot(ri[q] < 0);
    const int k = __popcll(fr & below);
    const int one = ri[q] < 0 && k < unit ? kLuNb - unit + k : -1;
    unit -= min(unit, (int)__popcll(fr));
    step[q] = ri[q] >= 0 || one >= 0 ? -1 : kLuNb;
#pragma unroll
    for (int g = 0; g < kLuNb / 4; ++g) {
      const Quad<T> x = *reinterpret_cast<const Quad<T> *>(P + max(min(s, cnt - 1), 0) * LS + 4 * g);
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2)
        v[q][4 * g + k2] = ri[q] >= 0 ? x.v[k2] : 4 * g + k2 == one ? (T)1 : (T)0;
    }
  }
  const int f = lu_panel<T, R>(v, step);
  if (f) return -1 - (p0 + f - 1);
  int pl = p;   // the first panel whose columns a pivot row of this panel has factors in
  int base = 0, need = hinext - hi, next = hi;   // dense: rows kept so far; banded: rows still to place
  int last = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int s = q * 64 + lane;
    const bool pivot = ri[q] >= 0 && step[q] >= 0, kept = ri[q] >= 0 && !pivot;
    if (ri[q] >= 0) {
      T *row16 = A + ri[q] * ld + p0;
#pragma unroll
      for (int g = 0; g < kLuNb / 4; ++g) {
        Quad<T> x;
#pragma unroll
        for (int k = 0; k < 4; ++k) x.v[k] = v[q][4 * g + k];
        *reinterpret_cast<Quad<T> *>(row16 + 4 * g) = x;
      }
    }
    if (pivot && step[q] < w) {   // (a failing panel may give a row a step past the last)
      perm[p0 + step[q]] = ri[q];
      L.piv(p)[step[q]] = ri[q];
      if (BAND) pl = min(pl, L.entry()[s]);
    }
    int slot, occupant = kept ? ri[q] : -1;
    bool store;
    if constexpr (BAND) {
      // a free slot takes the next entering row, in slot order
      const bool open = !kept && s < L.nslot;
      const unsigned long long fr = __ballot(open);
      const int k = __popcll(fr & below);
      if (open && k < need) {
        occupant = next + k;
        L.entry()[s] = p + 1;
      }
      const int placed = min(need, (int)__popcll(fr));
      need -= placed;
      next += placed;
      slot = s;
      store = s < L.nslot;
      const unsigned long long occ = __ballot(occupant >= 0);
      if (occ) last = q * 64 + 64 - __clzll(occ);
    } else {
      const unsigned long long kb = __ballot(kept);
      slot = base + __popcll(kb & below);
      base += __popcll(kb);
      last = base;
      store = kept;
    }
    if (store) {
      rown[slot] = occupant;
#pragma unroll
      for (int g = 0; g < kLuNb / 4; ++g) {
        Quad<T> x;
#pragma unroll
        for (int k = 0; k < 4; ++k) x.v[k] = kept ? v[q][4 * g + k] : (T)0;
        *reinterpret_cast<Quad<T> *>(P + slot * LS + 4 * g) = x;
      }
    }
  }
  if constexpr (BAND) {
    // the smallest entry panel over the pivot rows
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pl = min(pl, __shfl_xor(pl, o));
    if (lane == 0) plo[p] = pl;
  } else {
    // slots up to the end of the last tile: no row, no factor
    const int s = base + lane;
    if (lane < 16 && s < ((base + 15) & ~15)) {
      rown[s] = -1;
#pragma unroll
      for (int k = 0; k < kLuNb; ++k) P[s * LS + k] = 0;
    }
  }
  return last;
}

// Factors one matrix (n x n, leading dimension ld a multiple of 16 with the
// columns [n, ld) zero; base 16-byte aligned).  Banded: rows sorted by their
// first column; before panel p the rows [0, hi[p]) may be nonzero in its
// columns, and their last column is below cend[p]; at most nslot rows wait at
// a time.  nslot: slots in LDS, a multiple of 16.
template <typename T, int RMAX, bool BAND>
__device__ void lu_matrix(T *__restrict__ A, int n, int64_t ld, const int *__restrict__ hi,
                          const int *__restrict__ cend, int nslot, int *__restrict__ perm, int *__restrict__ plo,
                          int *__restrict__ status, unsigned char *lds) {
  typedef Mfma16<T> MM;
  typedef typename MM::acc acc;
  constexpr int LS = kLuStride<T>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jl = lane & 15, kq = lane >> 4;
  LuLds<T> L;
  L.base = reinterpret_cast<T *>(lds);
  L.ints = reinterpret_cast<int *>(L.base + 2 * nslot * LS);
  L.nslot = nslot;
  const int np = (n + kLuNb - 1) / kLuNb;
  int cnt = BAND ? hi[0] : n;
  for (int s = tid; s < nslot; s += kLuThreads) {
    L.row(0)[s] = s < cnt ? s : -1;
    L.row(1)[s] = -1;
    L.entry()[s] = 0;
  }
  __syncthreads();
  int fail = 0;
  for (int p = 0; p < np; ++p) {
    const int p0 = p * kLuNb, w = min(kLuNb, n - p0);
    const T *F = L.panel(p + 1);   // the previous panel's factors, in this panel's slots
    T *P = L.panel(p);
    const int *row = L.row(p);
    const int *piv = L.piv(p + 1);
    const int nrt = (cnt + 15) >> 4;
    // operands of the previous panel's update of 16 columns from c0: its
    // pivot rows there, as the k index runs over a lane's registers
    auto load_x = [&](int c0, T (&bx)[4]) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) bx[kk] = A[piv[4 * kq + kk] * ld + c0 + jl];
    };
    auto load_c = [&](int rt, int c0) {
      acc c;
#pragma unroll
      for (int r = 0; r < 4; ++r) c[r] = A[max(row[rt * 16 + MM::row(r, kq)], 0) * ld + c0 + jl];
      return c;
    };
    auto update = [&](int rt, const T (&bx)[4], acc c) {
      const Quad<T> a = *reinterpret_cast<const Quad<T> *>(F + (rt * 16 + jl) * LS + 4 * kq);
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) c = MM::mma(a.v[kk], bx[kk], c);
      return c;
    };
    // this panel's columns, brought up to date, into LDS
    {
      T bx[4] = {0, 0, 0, 0};
      if (p) load_x(p0, bx);
      for (int rt = wave; rt < nrt; rt += kLuWaves) {
        acc c = load_c(rt, p0);
        if (p) c = update(rt, bx, c);
#pragma unroll
        for (int r = 0; r < 4; ++r) P[(rt * 16 + MM::row(r, kq)) * LS + jl] = c[r];
      }
    }
    __syncthreads();
    if (wave == 0) {
      const int h0 = BAND ? hi[p] : n, h1 = BAND ? (p + 1 < np ? hi[p + 1] : h0) : n;
      int res = 0;
      // as few rows a lane as hold the slots in use, before and after
      const int rr = (min(nslot, cnt + (BAND ? h1 - h0 : 0)) + 63) >> 6;
#define FSI_LU_CASE(R) \
  if constexpr (R <= RMAX) { \
    res = lu_factor<T, R, BAND>(A, ld, p, w, cnt, h0, h1, L, perm, plo); \
  }
      if (rr <= 1) { FSI_LU_CASE(1) }
      else if (rr == 2) { FSI_LU_CASE(2) }
      else if (rr == 3) { FSI_LU_CASE(3) }
      else if (rr == 4) { FSI_LU_CASE(4) }
      else if (rr == 5) { FSI_LU_CASE(5) }
      else if (rr == 6) { FSI_LU_CASE(6) }
      else if (rr <= 9) { FSI_LU_CASE(9) }
      else { FSI_LU_CASE(13) }
#undef FSI_LU_CASE
      if (lane == 0) *L.result(p) = res;
    } else if (p) {
      // the previous panel's update of the columns beyond this panel: whole
      // 16-column tiles per wave, kLuAhead C tiles in flight
      const int ce = BAND ? cend[p - 1] : n;
      const int nct = (ce - p0 - 1) >> 4;   // tiles that start in [p0 + 16, ce)
      for (int ct = wave - 1; ct < nct; ct += kLuWaves - 1) {
        const int c0 = p0 + 16 + 16 * ct;
        T bx[4];
        load_x(c0, bx);
        acc ring[kLuAhead];
#pragma unroll
        for (int u = 0; u < kLuAhead; ++u) ring[u] = load_c(min(u, nrt - 1), c0);
        for (int rt0 = 0; rt0 < nrt; rt0 += kLuAhead) {
#pragma unroll
          for (int u = 0; u < kLuAhead; ++u) {
            const int rt = rt0 + u;
            if (rt < nrt) {
              const acc c = update(rt, bx, ring[u]);
              ring[u] = load_c(min(rt + kLuAhead, nrt - 1), c0);
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int i = row[rt * 16 + MM::row(r, kq)];
                if (i >= 0) A[i * ld + c0 + jl] = c[r];
              }
            }
          }
        }
      }
    }
    __threadfence_block();
    __syncthreads();
    const int res = *L.result(p);
    if (res < 0) {
      fail = -res;   // 1 + the failing step
      break;
    }
    cnt = res;
  }
  if (tid == 0) status[0] = fail;
  // a failed matrix keeps a permutation inside it: what reads the factors
  // runs before the host reads the status
  if (fail)
    for (int i = tid; i < n; i += kLuThreads) perm[i] = i;
  __syncthreads();
}

// Equilibration of the coarsest operator's free block by powers of two (no
// rounding): kEquilSteps alternating passes take the square root of each
// row's largest scaled entry out of the row, then likewise for the columns.
// The dofs' equations differ by many orders (momentum, kinematics, continuity,
// mesh motion), and in the banded order one panel mixes them: unscaled, the
// inverse of a 16x4 coarsest operator was 6e2 times further from the exact
// one than the Gauss-Jordan chain's (which takes the fields one after the
// other); scaled it is as close, and 1e3 times closer for a time step's.
// er[r]: the row's exponent; cmax[k][c]: the column's largest exponent in pass
// k, biased (0: none yet); both start at zero.  One wave per row.
constexpr int kEquilBias = 8192;
__device__ __forceinline__ int half_floor(int x) { return x >> 1; }
// the column's exponent after the first `passes` passes
__device__ __forceinline__ int col_exp(const int *__restrict__ cmax, int n, int c, int passes) {
  int e = 0;
  for (int k = 0; k < passes; ++k) {
    const int m = cmax[k * n + c];
    if (m) e -= half_floor(m - kEquilBias);
  }
  return e;
}
__global__ __launch_bounds__(256) void k_equil(int n, const int *__restrict__ rowptr, const int *__restrict__ col,
                                               const double *__restrict__ val, const int *__restrict__ fpos, int pass,
                                               int *__restrict__ er, int *__restrict__ cmax) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= n || fpos[r] < 0) return;
  // exponent of an entry of F with its scales (INT_MIN: zero or not finite)
  auto exponent = [&](int p, int e0) {
    const int b = (int)((__double_as_longlong(val[p]) >> 52) & 0x7ff);
    if (b == 0 || b == 0x7ff || fpos[col[p]] < 0) return INT_MIN;
    return b - 1022 + e0 + col_exp(cmax, n, col[p], pass);
  };
  int e0 = er[r], m = INT_MIN;
  const int p0 = rowptr[r], p1 = rowptr[r + 1];
  for (int p = p0 + lane; p < p1; p += 64) m = max(m, exponent(p, e0));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
  if (m == INT_MIN) return;
  e0 -= half_floor(m);
  if (lane == 0) er[r] = e0;
  for (int p = p0 + lane; p < p1; p += 64) {
    const int e = exponent(p, e0);
    if (e != INT_MIN) atomicMax(&cmax[pass * n + col[p]], e + kEquilBias);
  }
}

// the scaled free block into its ordered places (zero-filled beforehand); one
// wave per row
__global__ __launch_bounds__(256) void k_band_dense(int n, int64_t ld, const int *__restrict__ rowptr,
                                                    const int *__restrict__ col, const double *__restrict__ val,
                                                    const int *__restrict__ rpos, const int *__restrict__ cpos,
                                                    const int *__restrict__ er, const int *__restrict__ cmax,
                                                    double *__restrict__ A) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= n || rpos[r] < 0) return;
  for (int p = rowptr[r] + (threadIdx.x & 63); p < rowptr[r + 1]; p += 64) {
    const int c = cpos[col[p]];
    if (c >= 0) A[rpos[r] * ld + c] = ldexp(val[p], er[r] + col_exp(cmax, n, col[p], kEquilSteps));
  }
}

// banded coarsest operator: one workgroup (one compute unit of the device,
// beside the blocks' inversion)
template <int RMAX>
__global__ __launch_bounds__(kLuThreads) void k_lu_band(double *__restrict__ A, int n, int64_t ld,
                                                        const int *__restrict__ hi, const int *__restrict__ cend,
                                                        int nslot, int *__restrict__ perm, int *__restrict__ plo,
                                                        int *__restrict__ status) {
  extern __shared__ __align__(16) unsigned char lu_lds[];
  lu_matrix<double, RMAX, true>(A, n, ld, hi, cend, nslot, perm, plo, status, lu_lds);
}

// Rows of the inverse from the factors.  z A = e_i for 16 G unknowns i at a
// time (one right-hand side each): first w U = e_i panel by panel from the
// one that holds the first unknown, w_p = rhs_p B_p^-1, rhs_j -= w_p A[R_p][j]
// for the later panels j; then from the last panel down z = w, w_j += z_p
// PC[R_p][j] for the earlier ones.  Both directions use the tiles
// A[perm[16 p + k]][16 j + i] alike.  The right-hand sides sit in registers,
// tile j (16 entries of 16 G vectors) in wave j mod 8, so a panel costs one
// LDS broadcast of its 16 x 16 G values and one barrier; the values keep the
// layout of a product's result, which is that of its second operand when the
// k index of register r is MM::row(r, kq).  The wave that owns the next panel
// brings that tile up to date first and broadcasts it before its other tiles;
// a panel's factor tiles are loaded one panel ahead (TA of a wave's tiles;
// when more are in reach, the others are loaded where they are used).
// jlo(p): the first panel whose columns hold factors of panel p's rows;
// jhi(p): the end of the panels that its pivot rows reach.  prow: perm in
// LDS, 16 np entries, clamped to n - 1.  The entries past n of every vector
// are zero throughout (the matrix's columns past n are), so the clamped rows
// contribute nothing.
template <typename T, int TPW, int TA, int G, class JLo, class JHi>
__device__ __forceinline__ void lu_rows(const T *__restrict__ A, int n, int ld, const int *prow,
                                        const int (&pos)[G], int pstart, JLo jlo, JHi jhi, T *bc,
                                        typename Mfma16<T>::acc (&x)[TPW][G]) {
  typedef Mfma16<T> MM;
  typedef typename MM::acc acc;
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int np = (n + kLuNb - 1) / kLuNb;
#pragma unroll
  for (int u = 0; u < TPW; ++u)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        x[u][g][r] = pos[g] == (wave + kLuWaves * u) * kLuNb + MM::row(r, kq) ? (T)1 : (T)0;
  // offsets of this lane's entries in the pivot rows of panel p
  auto row_offsets = [&](int p, int (&ro)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) ro[kk] = prow[p * kLuNb + MM::row(kk, kq)] * ld + jl;
  };
  auto load_a = [&](const int (&ro)[4], int j, T (&a)[4]) {
    const T *Aj = A + j * kLuNb;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a[kk] = Aj[ro[kk]];
  };
  // the tiles [j0, j1) of this wave, the first TA of them, for panel p
  auto load_tiles = [&](int p, int j0, int j1, T (&a)[TA][4]) {
    const int u0 = max(j0 - wave + kLuWaves - 1, 0) / kLuWaves;
    int ro[4];
    row_offsets(p, ro);
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int j = wave + kLuWaves * u;
      if (j >= j0 && j < j1 && u - u0 < TA) load_a(ro, j, a[u % TA]);
    }
  };
  auto publish = [&](int p, const acc (&y)[G]) {
    T *b = bc + (p & 1) * G * 256;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) b[(g * 4 + r) * 64 + lane] = y[g][r];
  };
  auto fetch = [&](int p, acc (&y)[G]) {
    const T *b = bc + (p & 1) * G * 256;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[g][r] = b[(g * 4 + r) * 64 + lane];
  };
  auto apply = [&](const T (&a)[4], const acc (&y)[G], acc (&z)[G]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int g = 0; g < G; ++g) z[g] = MM::mma(a[kk], y[g][kk], z[g]);
  };
  // tile u of this wave (panel j) by panel p, whose tiles in reach start at j0
  auto apply_tile = [&](int u, int p, int j0, const T (&a)[TA][4], const acc (&y)[G]) {
    const int u0 = max(j0 - wave + kLuWaves - 1, 0) / kLuWaves;
    if (TA == TPW || u - u0 < TA) {
      apply(a[u % TA], y, x[u]);
    } else {
      T b[4];
      int ro[4];
      row_offsets(p, ro);
      load_a(ro, wave + kLuWaves * u, b);
      apply(b, y, x[u]);
    }
  };
  // w_p from the finished right-hand side of this wave's tile u, broadcast
  // with the sign that the later panels' updates take
  T ad[4];   // B^-1 of this wave's next panel
  auto finish = [&](int u, int p) {
    acc y[G];
#pragma unroll
    for (int g = 0; g < G; ++g) y[g] = acc{0, 0, 0, 0};
    apply(ad, x[u], y);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      x[u][g] = y[g];
      y[g] = -y[g];
    }
    publish(p, y);
    if (p + kLuWaves < np) {
      int ro[4];
      row_offsets(p + kLuWaves, ro);
      load_a(ro, p + kLuWaves, ad);
    }
  };
  // with registers to spare the next panel's tiles are loaded during this
  // one's products, else after them
  constexpr bool kAhead = TPW <= 9;
  T a[TA][4], an[kAhead ? TA : 1][4];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) a[i][k] = 0;
  auto take_next = [&] {
    if constexpr (kAhead) {
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) a[i][k] = an[i][k];
    }
  };
  {
    const int own = pstart + ((wave - pstart) & (kLuWaves - 1));   // this wave's first panel
    if (own < np) {
      int ro[4];
      row_offsets(own, ro);
      load_a(ro, own, ad);
    }
  }
  int jh = min(jhi(pstart), np);
  load_tiles(pstart, pstart + 1, jh, a);
#pragma unroll
  for (int u = 0; u < TPW; ++u)
    if (wave + kLuWaves * u == pstart) finish(u, pstart);
  for (int p = pstart; p + 1 < np; ++p) {
    const int jhn = min(jhi(p + 1), np);
    __syncthreads();
    acc y[G];
    fetch(p, y);
    if (wave == ((p + 1) & (kLuWaves - 1))) {
#pragma unroll
      for (int u = 0; u < TPW; ++u)
        if (wave + kLuWaves * u == p + 1) {
          if (p + 1 < jh) apply_tile(u, p, p + 1, a, y);
          finish(u, p + 1);
        }
    }
    if constexpr (kAhead)
      if (p + 2 < np) load_tiles(p + 1, p + 2, jhn, an);
#pragma unroll
    for (int u = 0; u < TPW; ++u)
      if (wave + kLuWaves * u > p + 1 && wave + kLuWaves * u < jh) apply_tile(u, p, p + 1, a, y);
    jh = jhn;
    if constexpr (!kAhead)
      if (p + 2 < np) load_tiles(p + 1, p + 2, jhn, a);
    take_next();
  }
  __syncthreads();   // the broadcast buffers are reused from the last panel down
  int j0 = jlo(np - 1);
  load_tiles(np - 1, j0, np - 1, a);
#pragma unroll
  for (int u = 0; u < TPW; ++u)
    if (wave + kLuWaves * u == np - 1) publish(np - 1, x[u]);
  for (int p = np - 1; p > 0; --p) {
    const int j0n = jlo(p - 1);
    __syncthreads();
    acc y[G];
    fetch(p, y);
    if (wave == ((p - 1) & (kLuWaves - 1))) {
#pragma unroll
      for (int u = 0; u < TPW; ++u)
        if (wave + kLuWaves * u == p - 1) {
          if (p - 1 >= j0) apply_tile(u, p, j0, a, y);
          publish(p - 1, x[u]);
        }
    }
    if constexpr (kAhead)
      if (p > 1) load_tiles(p - 1, j0n, p - 1, an);
#pragma unroll
    for (int u = 0; u < TPW; ++u)
      if (wave + kLuWaves * u < p - 1 && wave + kLuWaves * u >= j0) apply_tile(u, p, j0, a, y);
    j0 = j0n;
    if constexpr (!kAhead)
      if (p > 1) load_tiles(p - 1, j0n, p - 1, a);
    take_next();
  }
}

// The coarsest operator's inverse on its free block: workgroup b finds the
// rows of 16 consecutive columns of the ordered matrix and writes them to
// C0 (n0 x n0 row-major) at the dofs coldof (ordered columns) and rowdof
// (ordered rows) stand for, the equilibration undone.
template <int TPW, int TA>
__global__ __launch_bounds__(kLuThreads) void k_lu_band_rows(const double *__restrict__ A, int n, int ld,
                                                             const int *__restrict__ perm,
                                                             const int *__restrict__ plo,
                                                             const int *__restrict__ cend,
                                                             const int *__restrict__ status,
                                                             const int *__restrict__ rowdof,
                                                             const int *__restrict__ coldof,
                                                             const int *__restrict__ er,
                                                             const int *__restrict__ cmax, int n0,
                                                             double *__restrict__ C0) {
  typedef Mfma16<double> MM;
  __shared__ double bc[2 * 256];
  __shared__ int prow[TPW * kLuWaves * kLuNb];
  if (status[0]) return;
  for (int s = threadIdx.x; s < TPW * kLuWaves * kLuNb; s += kLuThreads) prow[s] = perm[min(s, n - 1)];
  __syncthreads();
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x;
  const int pos[1] = {b * kLuNb + jl};
  dx4 x[TPW][1];
  lu_rows<double, TPW, TA, 1>(
      A, n, ld, prow, pos, b, [&](int p) { return plo[p]; }, [&](int p) { return (cend[p] + kLuNb - 1) / kLuNb; },
      bc, x);
  if (pos[0] >= n) return;
  const int k = coldof[pos[0]], ec = col_exp(cmax, n0, k, kEquilSteps);
  double *C = C0 + (int64_t)k * n0;
#pragma unroll
  for (int u = 0; u < TPW; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int s = (wave + kLuWaves * u) * kLuNb + MM::row(r, kq);
      if (s < n) {
        const int c = rowdof[prow[s]];
        C[c] = ldexp(x[u][0][r], ec + er[c]);
      }
    }
}

// C0 outside the free block: 1 / a_dd on the diagonal of D, zero elsewhere
__global__ __launch_bounds__(256) void k_coarse_border(int n, const int *__restrict__ fpos,
                                                       const int *__restrict__ rowptr,
                                                       const double *__restrict__ val, double *__restrict__ C0) {
  const int c = blockIdx.x * 256 + threadIdx.x, k = blockIdx.y;
  if (c >= n || (fpos[k] >= 0 && fpos[c] >= 0)) return;
  C0[(int64_t)k * n + c] = k == c ? 1.0 / val[rowptr[k]] : 0.0;
}

template <int RMAX>
static void launch_band_factor(double *A, const BandView &B, int64_t ld, int *status, hipStream_t st) {
  const size_t shm = lu_lds_bytes(B.nslot, sizeof(double), kLuStride<double>);
  k_lu_band<RMAX><<<1, kLuThreads, shm, st>>>(A, B.n, ld, B.hi, B.cend, B.nslot, B.perm, B.plo, status);
}
template <int TPW, int TA>
static void launch_band_rows(const double *A, const BandView &B, int64_t ld, const int *status, int n0, double *C0,
                             hipStream_t st) {
  k_lu_band_rows<TPW, TA><<<(B.n + kLuNb - 1) / kLuNb, kLuThreads, 0, st>>>(A, B.n, (int)ld, B.perm, B.plo, B.cend, status,
                                                                       B.rowdof, B.coldof, B.scale, B.scale + n0, n0,
                                                                       C0);
}

template <int RMAX>
static void allow_band_lds() {
  (void)hipFuncSetAttribute((const void *)k_lu_band<RMAX>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lu_lds_bytes(64 * RMAX, sizeof(double), kLuStride<double>));
}
void lu_coarse_prepare() {
  static std::once_flag once;   // setup threads may come together
  std::call_once(once, [] {
    allow_band_lds<2>();
    allow_band_lds<4>();
    allow_band_lds<5>();
  });
}

void lu_coarse(double *A, int64_t ld, const BandView &B, const CsrView<double> &J, const CoarseSplit &cs, double *C0,
               int *status, hipStream_t st) {
  int *er = B.scale, *cmax = B.scale + cs.n;
  const int wg = (cs.n + 3) / 4;
  launch_fill_i32(B.scale, (kEquilSteps + 1) * cs.n, 0, st);
  for (int k = 0; k < kEquilSteps; ++k)
    k_equil<<<wg, 256, 0, st>>>(cs.n, J.rowptr, J.col, J.val, cs.fpos, k, er, cmax);
  launch_fill_f64(A, (int64_t)B.n * ld, 0.0, st);
  k_band_dense<<<wg, 256, 0, st>>>(cs.n, ld, J.rowptr, J.col, J.val, B.rpos, B.cpos, er, cmax, A);
  if (B.nslot <= 128)
    launch_band_factor<2>(A, B, ld, status, st);
  else if (B.nslot <= 256)
    launch_band_factor<4>(A, B, ld, status, st);
  else
    launch_band_factor<5>(A, B, ld, status, st);
  const int np = (B.n + kLuNb - 1) / kLuNb, tpw = (np + kLuWaves - 1) / kLuWaves;
  if (tpw <= 4)
    launch_band_rows<4, 4>(A, B, ld, status, cs.n, C0, st);
  else if (tpw <= 9)
    launch_band_rows<9, 4>(A, B, ld, status, cs.n, C0, st);
  else
    launch_band_rows<20, 3>(A, B, ld, status, cs.n, C0, st);
  launch_coarse_diagonal(cs, B.n, status, st);
  k_coarse_border<<<dim3((cs.n + 255) / 256, cs.n), 256, 0, st>>>(cs.n, cs.fpos, cs.rowptr, cs.val, C0);
}

}  // namespace fsi
