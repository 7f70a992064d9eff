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
#include <hip/hip_bf16.h>
#include <hip/hip_ext.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <climits>
#include <type_traits>

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

// Between one lane's LDS access and another lane's of the same wave.  The
// hardware keeps a wave's LDS operations in order; this keeps the compiler's
// (no instruction).
__device__ __forceinline__ void lu_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// the pivot row (lane ll, register row ql) into scalars
template <typename T, int R, int NC, int Q = 0>
__device__ __forceinline__ void lu_take(const T (&v)[R][NC], int ql, int ll, T (&prow)[NC]) {
  if (Q == R - 1 || ql == Q) {
#pragma unroll
    for (int c = 0; c < NC; ++c) prow[c] = readlane(v[Q][c], ll);
  } else if constexpr (Q + 1 < R) {
    lu_take<T, R, NC, Q + 1>(v, ql, ll, prow);
  }
}

// |a| as an unsigned integer: its bits (FP64: the upper half, 21 significant
// bits); at least kLuInf: infinite or no number
__device__ __forceinline__ unsigned lu_key(double a) {
  return (unsigned)(__double_as_longlong(a) >> 32) & 0x7fffffffu;
}
__device__ __forceinline__ unsigned lu_key(float a) { return __float_as_uint(a) & 0x7fffffffu; }
template <typename T>
constexpr unsigned kLuInf = sizeof(T) == 8 ? 0x7ff00000u : 0x7f800000u;
// wave-wide maximum (all lanes active), the same value in every lane
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned lu_dpp_max(unsigned v) {
  return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, ROWS == 0xF));
}
__device__ __forceinline__ unsigned lu_wave_max(unsigned v) {
  v = lu_dpp_max<kDppXor1, 0xF>(v);
  v = lu_dpp_max<kDppXor2, 0xF>(v);
  v = lu_dpp_max<kDppRor4, 0xF>(v);
  v = lu_dpp_max<kDppRor8, 0xF>(v);
  v = lu_dpp_max<kDppBcast15, 0xA>(v);
  v = lu_dpp_max<kDppBcast31, 0xC>(v);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// The pivot steps on columns t, t + 1, ... of a group of NC (see lu_columns);
// t0: the group's first step in the panel.  The pivot is the first lane's
// whose key is the largest: within 2^-20 of the largest candidate in FP64,
// which the growth of the factors does not feel, and one 32-bit maximum a
// reduction step instead of a 64-bit one with the row in it.  The next pivot
// column is eliminated first, so its search runs beside the other columns.
template <typename T, int R, int NC, int t>
__device__ __forceinline__ void lu_steps(T (&v)[R][NC], int (&step)[R], int t0, T *scale, int &fail) {
  const int lane = threadIdx.x & 63;
  unsigned key = 0;
  int lq = 0;
  T sv = 1;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const unsigned kq = step[q] < 0 ? lu_key(v[q][t]) : 0u;
    const bool more = kq > key;
    key = more ? kq : key;
    sv = more ? v[q][t] : sv;
    lq = more ? q : lq;
  }
  const T dl = recip(sv);   // every lane inverts its own candidate during the reduction
  const unsigned best = lu_wave_max(key);
  const bool bad = best == 0 || best >= kLuInf<T>;
  fail = fail == 0 && bad ? t0 + t + 1 : fail;
  const int ll = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(__ballot(key == best)));
  const int ql = R == 1 ? 0 : __builtin_amdgcn_readlane(lq, ll);
  const int slot = ql * 64 + ll;
  const T d = readlane(dl, ll);
  if (lane == 0) scale[t] = d;
  T prow[NC];
  lu_take<T, R, NC>(v, ql, ll, prow);
  T fd[R];
  bool own[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    own[q] = slot == q * 64 + lane;
    fd[q] = own[q] ? (T)0 : v[q][t] * d;
    step[q] = own[q] ? t0 + t : step[q];
  }
#pragma unroll
  for (int cc = 0; cc < NC; ++cc) {
    const int c = (t + 1 + cc) % NC;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      v[q][c] = c == t ? (own[q] ? (T)1 : -fd[q]) : v[q][c] - fd[q] * prow[c];
      // keeps each step's work in the step: deferred, the columns that no
      // later step searches would hold every pivot row in scalars to the end
      asm volatile("" : "+v"(v[q][c]));
    }
  }
  if constexpr (t + 1 < NC) lu_steps<T, R, NC, t + 1>(v, step, t0, scale, fail);
}

// Shared memory of a factorization: by the parity of a panel its rows (first
// the panel being factored, then its factors for the updates), the matrix row
// in each slot or -1, the panel's pivot rows in step order and the slots in
// use or the failure; (banded) the panel at which each slot's row entered; the
// factoring wave's reciprocals and pivot slots.  PB: panel buffers (one where
// the updates read the factors from the matrix).
template <typename T, int PB>
struct LuLds {
  T *base;
  int nslot;
  __device__ __forceinline__ T *panel(int p) const { return base + (p & (PB - 1)) * nslot * kLuStride<T>; }
  __device__ __forceinline__ T *scale() const { return base + PB * nslot * kLuStride<T>; }
  __device__ __forceinline__ int *ints() const { return reinterpret_cast<int *>(scale() + kLuNb); }
  __device__ __forceinline__ int *row(int p) const { return ints() + (p & 1) * nslot; }
  __device__ __forceinline__ int *entry() const { return ints() + 2 * nslot; }
  __device__ __forceinline__ int *piv(int p) const { return ints() + 3 * nslot + (p & 1) * kLuNb; }
  __device__ __forceinline__ int *slots() const { return ints() + 3 * nslot + 2 * kLuNb; }
  __device__ __forceinline__ int *result(int p) const { return ints() + 3 * nslot + 3 * kLuNb + (p & 1); }
};
template <typename T>
static inline size_t lu_lds_bytes(int nslot, int pb) {
  return sizeof(T) * ((size_t)pb * nslot * kLuStride<T> + kLuNb) + sizeof(int) * (3 * (size_t)nslot + 3 * kLuNb + 2);
}

// (No variant may spill: once the compiler put the spills of a lane's slot
// rows into one side of a divergent branch, and the lanes of the other side
// later stored to rows read from stale scratch memory.)
// Columns [c0, c0 + NC) of the panel at P factored by one wave.  Lane l holds
// the rows of slots l + 64 q in registers; step[q] is -1 for a row that waits
// for its pivot (a candidate) and becomes the step at which it is the pivot,
// other slots have a step >= 16 and take no part.  Every row is eliminated in every
// column of the group (Gauss-Jordan inside it); a pivot row stays unscaled
// until the end (1 in its own column, and it takes the later eliminations like
// any other), so that a step has no branch that moves rows between registers.
// Returns 0, or 1 + the first step whose pivot is zero or not finite (the
// steps go on without a branch; the result is unusable).
template <typename T, int R, int NC, int PB>
__device__ __forceinline__ int lu_columns(T *P, int c0, int (&step)[R], const LuLds<T, PB> &L) {
  constexpr int LS = kLuStride<T>;
  const int lane = threadIdx.x & 63;
  T v[R][NC];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const bool use = step[q] < kLuNb;
    const T *x = P + (use ? q * 64 + lane : 0) * LS + c0;
#pragma unroll
    for (int g = 0; g < NC / 4; ++g) {
      const Quad<T> y = *reinterpret_cast<const Quad<T> *>(x + 4 * g);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[q][4 * g + k] = use ? y.v[k] : (T)0;
    }
  }
  int fail = 0;
  lu_steps<T, R, NC, 0>(v, step, c0, L.scale(), fail);
  lu_wave_sync();   // lane 0's reciprocals
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const bool pivot = step[q] >= c0 && step[q] < c0 + NC;
    const T sc = pivot ? L.scale()[step[q] - c0] : (T)1;
    if (pivot) L.slots()[step[q]] = q * 64 + lane;
    if (step[q] < kLuNb) {
      T *x = P + (q * 64 + lane) * LS + c0;
#pragma unroll
      for (int g = 0; g < NC / 4; ++g) {
        Quad<T> y;
#pragma unroll
        for (int k = 0; k < 4; ++k) y.v[k] = v[q][4 * g + k] * sc;
        *reinterpret_cast<Quad<T> *>(x + 4 * g) = y;
      }
    }
  }
  return fail;
}

// A factored group of NC columns applied to the panel's other columns (one
// wave, on the matrix cores, in LDS): row i takes sum_t PC[i][t] X[t], X the
// group's pivot rows before the update, which start from zero.
template <typename T, int NC, int PB>
__device__ __forceinline__ void lu_cross(T *P, int c0, int nrt, const LuLds<T, PB> &L) {
  typedef Mfma16<T> MM;
  typedef typename MM::acc acc;
  constexpr int LS = kLuStride<T>, KK = NC / 4;
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const bool other = jl < c0 || jl >= c0 + NC;
  const int *slots = L.slots() + c0;
  T bx[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const T x = P[slots[KK * kq + kk] * LS + jl];
    bx[kk] = other ? x : (T)0;
  }
  lu_wave_sync();   // every lane has its part of the pivot rows
#pragma unroll
  for (int t = 0; t < NC; t += 4)
    if (other) P[slots[t + kq] * LS + jl] = 0;
  lu_wave_sync();
  for (int rt = 0; rt < nrt; ++rt) {
    const T *a = P + (rt * 16 + jl) * LS + c0 + KK * kq;
    acc c;
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = P[(rt * 16 + MM::row(r, kq)) * LS + jl];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) c = MM::mma(a[kk], bx[kk], c);
#pragma unroll
    for (int r = 0; r < 4; ++r) P[(rt * 16 + MM::row(r, kq)) * LS + jl] = c[r];
  }
}

// The factoring wave's part of panel p: the rows of slots [0, cnt) in LDS
// (with the panel's columns up to date) factored in groups of NC columns (as
// many as its registers hold with R rows a lane), the factors to the matrix
// and to LDS, and the slots of the next panel.  Banded: a row keeps its slot
// until it is a pivot, freed slots go to the rows [hi, hinext) that enter
// next.  Dense: the rows left are moved together.  Returns the slots in use
// for the next panel, or -1 - step on a failing pivot.
template <typename T, int R, int NC, bool BAND, int PB>
__device__ __forceinline__ int lu_factor(T *__restrict__ A, int64_t ld, int p, int w, int cnt, int hi, int hinext,
                                         const LuLds<T, PB> &L, int *__restrict__ perm, int *__restrict__ plo) {
  constexpr int LS = kLuStride<T>;
  const int lane = threadIdx.x & 63, p0 = p * kLuNb;
  const unsigned long long below = (1ull << lane) - 1;
  T *P = L.panel(p);
  const int *row = L.row(p);
  int *rown = L.row(p + 1);
  int step[R];
  int unit = kLuNb - w;   // a last panel of w < 16 columns: the other pivots are unit rows in free slots
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int s = q * 64 + lane;
    const bool taken = s < cnt && row[s] >= 0, open = !taken && s < L.nslot;
    const unsigned long long fr = __ballot(open);
    const int k = __popcll(fr & below);
    const bool one = open && k < unit;
    if (one)
#pragma unroll
      for (int c = 0; c < kLuNb; ++c) P[s * LS + c] = c == kLuNb - unit + k ? (T)1 : (T)0;
    unit -= min(unit, (int)__popcll(fr));
    step[q] = taken || one ? -1 : kLuNb;
  }
  if (lane < kLuNb) L.slots()[lane] = 0;
  lu_wave_sync();
  int f = 0;
  if constexpr (NC == kLuNb) {
    f = lu_columns<T, R, NC, PB>(P, 0, step, L);
  } else {
    for (int c0 = 0; c0 < kLuNb; c0 += NC) {
      const int g = lu_columns<T, R, NC, PB>(P, c0, step, L);
      f = f ? f : g;
      lu_wave_sync();   // the group's rows and pivot slots
      lu_cross<T, NC, PB>(P, c0, (cnt + 15) >> 4, L);
      lu_wave_sync();
    }
  }
  if (f) return -1 - (p0 + f - 1);
  int pl = p;   // the first panel whose columns a pivot row of this panel has factors in
  int base = 0, need = hinext - hi, next = hi;   // dense: rows kept so far; banded: rows still to place
  int last = 0;
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int s = q * 64 + lane;
    const int ri = s < cnt ? row[s] : -1;
    const bool pivot = ri >= 0 && step[q] >= 0, kept = ri >= 0 && !pivot;
    Quad<T> x[kLuNb / 4];
#pragma unroll
    for (int g = 0; g < kLuNb / 4; ++g) {
      const Quad<T> y = *reinterpret_cast<const Quad<T> *>(P + (ri >= 0 ? s : 0) * LS + 4 * g);
#pragma unroll
      for (int k = 0; k < 4; ++k) x[g].v[k] = y.v[k];
      if (ri >= 0) *reinterpret_cast<Quad<T> *>(A + ri * ld + p0 + 4 * g) = x[g];
    }
    if (pivot && step[q] < w) {
      perm[p0 + step[q]] = ri;
      L.piv(p)[step[q]] = ri;
      if (BAND) pl = min(pl, L.entry()[s]);
    }
    int slot, occupant = kept ? ri : -1;
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
      // (slots below the ones read so far)
      const unsigned long long kb = __ballot(kept);
      slot = base + __popcll(kb & below);
      base += __popcll(kb);
      last = base;
      store = kept;
    }
    if constexpr (!BAND) lu_wave_sync();   // every lane has its row before another takes the slot
    if (store) {
      rown[slot] = occupant;
      if constexpr (PB == 2) {
#pragma unroll
        for (int g = 0; g < kLuNb / 4; ++g) {
#pragma unroll
          for (int k = 0; k < 4; ++k) x[g].v[k] = kept ? x[g].v[k] : (T)0;
          *reinterpret_cast<Quad<T> *>(P + slot * LS + 4 * g) = x[g];
        }
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
      if constexpr (PB == 2) {
#pragma unroll
        for (int k = 0; k < kLuNb; ++k) P[s * LS + k] = 0;
      }
    }
  }
  return last;
}

// Factors one matrix (n x n, leading dimension ld a multiple of 16 with the
// columns [n, ld) zero; base 16-byte aligned).  Banded: rows sorted by their
// first column; before panel p the rows [0, hi[p]) may be nonzero in its
// columns, and their last column is below cend[p]; at most nslot rows wait at
// a time, at least one before each panel (hi[p] > 16 p: BandOrder::full).
// nslot: slots in LDS, a multiple of 16.
template <typename T, int RMAX, bool BAND, int PB>
__device__ __forceinline__ void lu_matrix(T *__restrict__ A, int n, int64_t ld, const int *__restrict__ hi,
                          const int *__restrict__ cend, int nslot, int *__restrict__ perm, int *__restrict__ plo,
                          int *__restrict__ status, unsigned char *lds) {
  typedef Mfma16<T> MM;
  typedef typename MM::acc acc;
  constexpr int LS = kLuStride<T>;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jl = lane & 15, kq = lane >> 4;
  LuLds<T, PB> L;
  L.base = reinterpret_cast<T *>(lds);
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
    // the previous panel's factors of a tile's rows, from LDS or the matrix
    // (there the slots without a row repeat row 0; their results go nowhere)
    auto load_f = [&](int rt) {
      if constexpr (PB == 2)
        return *reinterpret_cast<const Quad<T> *>(F + (rt * 16 + jl) * LS + 4 * kq);
      else
        return *reinterpret_cast<const Quad<T> *>(A + max(row[rt * 16 + jl], 0) * ld + p0 - kLuNb + 4 * kq);
    };
    auto update = [&](const Quad<T> &a, const T (&bx)[4], acc c) {
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
        if (p) c = update(load_f(rt), bx, c);
#pragma unroll
        for (int r = 0; r < 4; ++r) P[(rt * 16 + MM::row(r, kq)) * LS + jl] = c[r];
      }
    }
    __syncthreads();
    if (wave == 0) {
      __builtin_amdgcn_s_setprio(3);   // the pivot chain before the updates that share its SIMD
      const int h0 = BAND ? hi[p] : n, h1 = BAND ? (p + 1 < np ? hi[p + 1] : h0) : n;
      int res = 0;
      // as few rows a lane as hold the slots in use, before and after
      const int rr = (min(nslot, cnt + (BAND ? h1 - h0 : 0)) + 63) >> 6;
#define FSI_LU_CASE(R, NC)                                                              \
  if constexpr (R <= RMAX) {                                                            \
    res = lu_factor<T, R, NC, BAND, PB>(A, ld, p, w, cnt, h0, h1, L, perm, plo);        \
  }
      // groups of as many columns as R rows a lane leave registers for
      constexpr bool kDouble = sizeof(T) == 8;
      if (rr <= 1) { FSI_LU_CASE(1, 16) }
      else if (rr == 2) { FSI_LU_CASE(2, 16) }
      else if (rr <= 4) { FSI_LU_CASE(4, 16) }
      else if (rr <= 6) { FSI_LU_CASE(6, (kDouble ? 8 : 16)) }
      else if (rr <= 8) { FSI_LU_CASE(8, (kDouble || RMAX > 8 ? 8 : 16)) }
      else { FSI_LU_CASE(13, 4) }
#undef FSI_LU_CASE
      if (lane == 0) *L.result(p) = res;
      __builtin_amdgcn_s_setprio(0);
    } else if (p) {
      // the previous panel's update of the columns beyond this panel: whole
      // 16-column tiles per wave, kLuAhead C tiles in flight
      const int ce = BAND ? cend[p - 1] : n;
      // tiles that start in [p0 + 16, ce); none without a row to update
      const int nct = nrt ? (ce - p0 - 1) >> 4 : 0;
      for (int ct = wave - 1; ct < nct; ct += kLuWaves - 1) {
        const int c0 = p0 + 16 + 16 * ct;
        T bx[4];
        load_x(c0, bx);
        // a tile's rows and factors are fetched with its values
        struct Tile {
          int r[4];
          Quad<T> f;
          acc c;
        } ring[kLuAhead];
        auto fetch = [&](int rt, Tile &t) {
#pragma unroll
          for (int r = 0; r < 4; ++r) t.r[r] = row[rt * 16 + MM::row(r, kq)];
          t.f = load_f(rt);
#pragma unroll
          for (int r = 0; r < 4; ++r) t.c[r] = A[max(t.r[r], 0) * ld + c0 + jl];
        };
#pragma unroll
        for (int u = 0; u < kLuAhead; ++u) fetch(min(u, nrt - 1), ring[u]);
        for (int rt0 = 0; rt0 < nrt; rt0 += kLuAhead) {
#pragma unroll
          for (int u = 0; u < kLuAhead; ++u) {
            const int rt = rt0 + u;
            if (rt < nrt) {
              Tile &t = ring[u];
              const acc c = update(t.f, bx, t.c);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (t.r[r] >= 0) A[t.r[r] * ld + c0 + jl] = c[r];
              fetch(min(rt + kLuAhead, nrt - 1), t);
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
// wave per row.  An entry that is not finite fails the operator here (status:
// 1 + its column's step): only the rows that wait together with its row take
// its column's update, so where the window empties no pivot would show it.
__global__ __launch_bounds__(256) void k_band_dense(int n, int64_t ld, const int *__restrict__ rowptr,
                                                    const int *__restrict__ col, const double *__restrict__ val,
                                                    const int *__restrict__ rpos, const int *__restrict__ cpos,
                                                    const int *__restrict__ er, const int *__restrict__ cmax,
                                                    double *__restrict__ A, int *__restrict__ status) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= n || rpos[r] < 0) return;
  for (int p = rowptr[r] + (threadIdx.x & 63); p < rowptr[r + 1]; p += 64) {
    const int c = cpos[col[p]];
    if (c < 0) continue;
    if (!(fabs(val[p]) <= DBL_MAX)) atomicMax(status, 1 + c);
    A[rpos[r] * ld + c] = ldexp(val[p], er[r] + col_exp(cmax, n, col[p], kEquilSteps));
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
  if (status[0]) return;   // an entry that is not finite
  lu_matrix<double, RMAX, true, 2>(A, n, ld, hi, cend, nslot, perm, plo, status, lu_lds);
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
// contribute nothing.  pos: this lane's unknown in each 16-vector tile (a
// negative one: none), the first ng <= G tiles hold any.
template <typename T, int TPW, int TA, int G, class JLo, class JHi>
__device__ __forceinline__ void lu_rows(const T *__restrict__ A, int n, int ld, const int *prow,
                                        const int (&pos)[G], int ng, int pstart, JLo jlo, JHi jhi, T *bc,
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
    for (int g = 0; g < G; ++g)
      if (g < ng) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) z[g] = MM::mma(a[kk], y[g][kk], z[g]);
      }
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
  constexpr bool kAhead = TPW * G * (int)sizeof(T) <= 96;
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
      if (wave + kLuWaves * u > p + 1 && wave + kLuWaves * u < jh) 
        apply_tile(u, p, p + 1, a, y);
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
      if (wave + kLuWaves * u < p - 1 && wave + kLuWaves * u >= j0) 
        apply_tile(u, p, j0, a, y);
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
  for (int s = threadIdx.x; s < TPW * kLuWaves * kLuNb; s += kLuThreads) prow[s] = min(max(perm[min(s, n - 1)], 0), n - 1);
  __syncthreads();
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x;
  const int pos[1] = {b * kLuNb + jl};
  dx4 x[TPW][1];
  lu_rows<double, TPW, TA, 1>(
      A, n, ld, prow, pos, 1, b, [&](int p) { return plo[p]; }, [&](int p) { return (cend[p] + kLuNb - 1) / kLuNb; },
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

// The same for a matrix of more panels than a wave holds tiles of.  Each wave
// keeps in registers the TPW of its tiles around the current panel: slot u is
// tile 8 (p / 8 + u) + wave going forward, 8 (p / 8 - u) + wave going back, and
// the slots move up by one every eight panels.  Forward no panel reaches
// further (the host has checked cend); back, a row that waited long has factors
// in panels before the window, whose tiles are then updated in memory.  A tile
// outside the window lies in its final place in C0, unscaled until z is final,
// and always by the same lanes; `kept` marks this wave's tiles that are there
// (the others are zero).  2,522 unknowns: 851 us, 178 registers; with all 20
// tiles of a wave in registers 1,485 of them spilled, 1,584 us.
template <int TPW, int TA>
__global__ __launch_bounds__(kLuThreads) void k_lu_band_rows_long(const double *__restrict__ A, int n, int ld,
                                                                  const int *__restrict__ perm,
                                                                  const int *__restrict__ plo,
                                                                  const int *__restrict__ cend,
                                                                  const int *__restrict__ status,
                                                                  const int *__restrict__ rowdof,
                                                                  const int *__restrict__ coldof,
                                                                  const int *__restrict__ er,
                                                                  const int *__restrict__ cmax, int n0, double *C0) {
  typedef Mfma16<double> MM;
  // a slot's preloaded factors keep their place when the slots move
  static_assert(TA + 2 <= TPW && TPW % TA == 0 && kLuBandMax <= 64 * kLuWaves * kLuNb, "");
  __shared__ double bc[2 * 256];
  __shared__ int prow[kLuBandMax];
  if (status[0]) return;
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x, np = (n + kLuNb - 1) / kLuNb;
  for (int s = threadIdx.x; s < np * kLuNb; s += kLuThreads) prow[s] = min(max(perm[min(s, n - 1)], 0), n - 1);
  __syncthreads();
  const bool mine = b * kLuNb + jl < n;   // this lane's unknown
  const int k = coldof[min(b * kLuNb + jl, n - 1)], ec = col_exp(cmax, n0, k, kEquilSteps);
  double *C = C0 + (int64_t)k * n0;
  auto load_a = [&](int p, int j, double (&a)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a[kk] = A[prow[p * kLuNb + MM::row(kk, kq)] * ld + j * kLuNb + jl];
  };
  auto apply = [&](const double (&a)[4], const dx4 &y, dx4 &z) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) z = MM::mma(a[kk], y[kk], z);
  };
  auto publish = [&](int p, const dx4 &y) {
#pragma unroll
    for (int r = 0; r < 4; ++r) bc[(p & 1) * 256 + r * 64 + lane] = y[r];
  };
  auto fetch = [&](int p) {
    dx4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = bc[(p & 1) * 256 + r * 64 + lane];
    return y;
  };
  uint64_t kept = 0;
  auto put = [&](int j, const dx4 &z, bool last) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int s = j * kLuNb + MM::row(r, kq);
      if (mine && s < n) {
        const int c = rowdof[prow[s]];
        C[c] = last ? ldexp(z[r], ec + er[c]) : z[r];
      }
    }
    kept |= 1ull << (j / kLuWaves);
  };
  auto get = [&](int j) {
    dx4 z = {0, 0, 0, 0};
    if (j >= 0 && ((kept >> (j / kLuWaves)) & 1)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = j * kLuNb + MM::row(r, kq);
        if (mine && s < n) z[r] = C[rowdof[prow[s]]];
      }
    }
    return z;
  };
  dx4 x[TPW];
  double a[TA][4], an[TA][4];
#pragma unroll
  for (int i = 0; i < TA; ++i)
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a[i][kk] = an[i][kk] = 0;
  // the slots moved up by one, the preloaded factors with them
  auto move = [&](const dx4 &in) {
#pragma unroll
    for (int u = 0; u + 1 < TPW; ++u) x[u] = x[u + 1];
    x[TPW - 1] = in;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const double t = a[0][kk];
#pragma unroll
      for (int i = 0; i + 1 < TA; ++i) a[i][kk] = a[i + 1][kk];
      a[TA - 1][kk] = t;
    }
  };
  auto take_next = [&] {
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) a[i][kk] = an[i][kk];
  };
  // tile j of slot u by panel p: its factors preloaded in the first TA slots from u0 on
  auto apply_slot = [&](int u, int u0, int p, int j, const dx4 &y) {
    if (u - u0 < TA) {
      apply(a[u % TA], y, x[u]);
    } else {
      double t[4];
      load_a(p, j, t);
      apply(t, y, x[u]);
    }
  };
  // forward: w_p from the finished right-hand side in slot u
  double ad[4] = {0, 0, 0, 0};   // B^-1 of this wave's next panel
  auto finish = [&](int u, int p) {
    dx4 y = {0, 0, 0, 0};
    apply(ad, x[u], y);
    put(p, y, false);
    publish(p, -y);
    if (p + kLuWaves < np) load_a(p + kLuWaves, p + kLuWaves, ad);
  };
  auto fwd_first = [&](int p, int v0) { return kLuWaves * v0 + wave > p ? 0 : kLuWaves * (v0 + 1) + wave > p ? 1 : 2; };
  auto fwd_load = [&](int p, int v0, int jh) {
    const int u0 = fwd_first(p, v0);
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int j = kLuWaves * (v0 + u) + wave;
      if (u >= u0 && u - u0 < TA && j < jh) load_a(p, j, an[u % TA]);
    }
  };
#pragma unroll
  for (int u = 0; u < TPW; ++u) x[u] = dx4{0, 0, 0, 0};
  if (wave == (b & (kLuWaves - 1)))
#pragma unroll
    for (int r = 0; r < 4; ++r) x[0][r] = jl == MM::row(r, kq) ? 1.0 : 0.0;
  {
    const int own = b + ((wave - b) & (kLuWaves - 1));   // this wave's first panel
    if (own < np) load_a(own, own, ad);
  }
  auto end_of = [&](int p) { return min((cend[p] + kLuNb - 1) / kLuNb, np); };
  int jh = end_of(b);
  fwd_load(b, b / kLuWaves, jh);
  take_next();
  if (wave == (b & (kLuWaves - 1))) finish(0, b);
  for (int p = b; p + 1 < np; ++p) {
    const int v0 = p / kLuWaves, jhn = end_of(p + 1);
    if (p > b && (p & (kLuWaves - 1)) == 0) move(dx4{0, 0, 0, 0});
    __syncthreads();
    const dx4 y = fetch(p);
    const int u0 = fwd_first(p, v0);
    if (wave == ((p + 1) & (kLuWaves - 1))) {
      if (wave) {
        if (p + 1 < jh) apply_slot(0, u0, p, p + 1, y);
        finish(0, p + 1);
      } else {
        if (p + 1 < jh) apply_slot(1, u0, p, p + 1, y);
        finish(1, p + 1);
      }
    }
    if (p + 2 < np) fwd_load(p + 1, v0, jhn);
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int j = kLuWaves * (v0 + u) + wave;
      if (j > p + 1 && j < jh) apply_slot(u, u0, p, j, y);
    }
    jh = jhn;
    take_next();
  }
  __syncthreads();   // the broadcast buffers are reused from the last panel down
  auto back_first = [&](int p, int v0) { return kLuWaves * v0 + wave < p ? 0 : kLuWaves * (v0 - 1) + wave < p ? 1 : 2; };
  auto back_load = [&](int p, int v0, int j0) {
    const int u0 = back_first(p, v0);
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int j = kLuWaves * (v0 - u) + wave;
      if (u >= u0 && u - u0 < TA && j >= j0) load_a(p, j, an[u % TA]);
    }
  };
  const int vl = (np - 1) / kLuWaves;
#pragma unroll
  for (int u = 0; u < TPW; ++u) x[u] = get(kLuWaves * (vl - u) + wave);
  int j0 = plo[np - 1];
  back_load(np - 1, vl, j0);
  take_next();
  if (wave == ((np - 1) & (kLuWaves - 1))) {
    put(np - 1, x[0], true);
    publish(np - 1, x[0]);
  }
  for (int p = np - 1; p > 0; --p) {
    const int v0 = p / kLuWaves, j0n = plo[p - 1];
    if (p < np - 1 && (p & (kLuWaves - 1)) == kLuWaves - 1) move(get(kLuWaves * (v0 - TPW + 1) + wave));
    __syncthreads();
    const dx4 y = fetch(p);
    const int u0 = back_first(p, v0);
    if (wave == ((p - 1) & (kLuWaves - 1))) {
      const int j = p - 1;
      if (wave != kLuWaves - 1) {
        if (j >= j0) apply_slot(0, u0, p, j, y);
        put(j, x[0], true);
        publish(j, x[0]);
      } else {
        if (j >= j0) apply_slot(1, u0, p, j, y);
        put(j, x[1], true);
        publish(j, x[1]);
      }
    }
    if (p > 1) back_load(p - 1, v0, j0n);
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
      const int j = kLuWaves * (v0 - u) + wave;
      if (j < p - 1 && j >= j0) apply_slot(u, u0, p, j, y);
    }
    for (int j = kLuWaves * (v0 - TPW) + wave; j >= j0; j -= kLuWaves) {
      dx4 z = get(j);
      double t[4];
      load_a(p, j, t);
      apply(t, y, z);
      put(j, z, false);
    }
    j0 = j0n;
    take_next();
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
  const size_t shm = lu_lds_bytes<double>(B.nslot, 2);
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
static hipError_t allow_band_lds() {
  static std::atomic<uint64_t> devices{0};
  return allow_lds(devices, (const void *)k_lu_band<RMAX>,
                   lu_lds_bytes<double>(std::min(64 * RMAX, kLuBandSlots), 2));
}
hipError_t lu_coarse_prepare(int nslot) {
  return nslot <= 128 ? allow_band_lds<2>() : nslot <= 256 ? allow_band_lds<4>() : allow_band_lds<6>();
}

// panels of which each wave keeps all its tiles (k_lu_band_rows)
constexpr int kLuBandResident = 9 * kLuWaves;
bool lu_band_reach_ok(const int *cend, int n) {
  const int np = (n + kLuNb - 1) / kLuNb;
  if (np <= kLuBandResident) return true;
  for (int p = 0; p < np; ++p)
    if ((cend[p] - 1) / kLuNb / kLuWaves - p / kLuWaves >= kLuBandWindow) return false;
  return true;
}

void lu_coarse(double *A, int64_t ld, const BandView &B, const CsrView<double> &J, const CoarseSplit &cs, double *C0,
               int *status, hipStream_t st) {
  int *er = B.scale, *cmax = B.scale + cs.n;
  const int wg = (cs.n + 3) / 4;
  launch_fill_i32(B.scale, (kEquilSteps + 1) * cs.n, 0, st);
  for (int k = 0; k < kEquilSteps; ++k)
    k_equil<<<wg, 256, 0, st>>>(cs.n, J.rowptr, J.col, J.val, cs.fpos, k, er, cmax);
  launch_fill_f64(A, (int64_t)B.n * ld, 0.0, st);
  k_band_dense<<<wg, 256, 0, st>>>(cs.n, ld, J.rowptr, J.col, J.val, B.rpos, B.cpos, er, cmax, A,
                                   status);
  if (B.nslot <= 128)
    launch_band_factor<2>(A, B, ld, status, st);
  else if (B.nslot <= 256)
    launch_band_factor<4>(A, B, ld, status, st);
  else
    launch_band_factor<6>(A, B, ld, status, st);
  const int np = (B.n + kLuNb - 1) / kLuNb;
  if (np <= 4 * kLuWaves)
    launch_band_rows<4, 4>(A, B, ld, status, cs.n, C0, st);
  else if (np <= kLuBandResident)
    launch_band_rows<9, 4>(A, B, ld, status, cs.n, C0, st);
  else
    k_lu_band_rows_long<kLuBandWindow, 4><<<np, kLuThreads, 0, st>>>(A, B.n, (int)ld, B.perm, B.plo, B.cend, status,
                                                                    B.rowdof, B.coldof, B.scale, B.scale + cs.n, cs.n,
                                                                    C0);
  launch_coarse_diagonal(cs, B.n, status, st);
  k_coarse_border<<<dim3((cs.n + 255) / 256, cs.n), 256, 0, st>>>(cs.n, cs.fpos, cs.rowptr, cs.val, C0);
}

// ------------------------------------------------------------------ Schwarz blocks
// Rows of a level's operator scaled by powers of two to a largest entry in
// [1/2, 1), for the extraction of its blocks: with the equations of both
// materials in one block, pivots chosen by unscaled magnitudes lose digits
// (a time step's interface block of 336 dofs: error of the inverse 9e-12, and
// 9e-14 scaled).  er: the rows' exponents.  One row per 16 lanes.
template <typename T>
__global__ __launch_bounds__(256) void k_scale_rows(int n, const int *__restrict__ rowptr,
                                                    const double *__restrict__ val, T *__restrict__ out,
                                                    int *__restrict__ er) {
  const int r = blockIdx.x * 16 + (threadIdx.x >> 4), sub = threadIdx.x & 15;
  if (r >= n) return;
  const int p0 = rowptr[r], p1 = rowptr[r + 1];
  int top = 0;   // the largest biased exponent of a finite entry
#pragma unroll 4
  for (int p = p0 + sub; p < p1; p += 16) {
    const int b = (int)((__double_as_longlong(val[p]) >> 52) & 0x7ff);
    top = max(top, b == 0x7ff ? 0 : b);
  }
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o));
  const int e = top ? 1022 - top : 0;
  if (sub == 0) er[r] = e;
#pragma unroll 4
  for (int p = p0 + sub; p < p1; p += 16) out[p] = (T)ldexp(val[p], e);
}

// One workgroup per block, the largest first.  Up to 372 dofs (336 blocks, more
// than compute units) it is bound by the updates' traffic: 4.9 GB in 1.11 ms in
// FP64, 4.4 TB/s, a plain copy's rate; one block alone takes 0.35 ms, the chain
// of pivot steps.  Larger blocks (one
// workgroup to a compute unit) are bound by that chain.
template <typename T, int RMAX, int PB>
__global__ __launch_bounds__(kLuThreads) void k_lu_blocks(T *__restrict__ blocks, const int64_t *__restrict__ boff,
                                                          const int *__restrict__ pm,
                                                          const int64_t *__restrict__ poff,
                                                          int *__restrict__ perm, int *__restrict__ status,
                                                          const int *__restrict__ order) {
  extern __shared__ __align__(16) unsigned char lu_lds[];
  const int k = order[blockIdx.x], m = pm[k], ld = block_ld(m);
  lu_matrix<T, RMAX, false, PB>(blocks + boff[k], m, ld, nullptr, nullptr, ld, perm + poff[k], nullptr, status + k,
                            lu_lds);
}

// Rows of the inverses in the Schwarz kernels' layout: one workgroup per task
// (a block, up to 64 rows of its inverse), written column by column (entry
// (c, r) of a task of nr rows at c nr + r), which is how the rows' 16-vector
// tiles come out: 16 rows of one column side by side in 16 lanes; the scales
// of the blocks' rows go into the inverse's columns.  cscale
// (with 16-bit storage): the largest magnitude of every column over the
// block's rows, as float bits.  The tasks of one XCD are consecutive, so a
// block's factors stay in its L2 for all of its tasks.
template <typename T, int TPW, int G>
__global__ __launch_bounds__(kLuThreads) void k_lu_rows(LuRowsBatch<T> B, int ntask, int chunk) {
  typedef Mfma16<T> MM;
  __shared__ T bc[2 * G * 256];
  __shared__ int prow[TPW * kLuWaves * kLuNb], scale[TPW * kLuWaves * kLuNb];
  const int task = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if (task >= ntask) return;
  int e = 0;
  while (e + 1 < B.count && task >= B.task0[e + 1]) ++e;
  const LuRowsItem<T> &it = B.it[e];
  const int t = task - B.task0[e];
  const int lane = threadIdx.x & 63, jl = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = it.task_patch[t], r0 = it.task_row0[t], m = it.pm[k];
  const int nr = min(64, it.po[k] - r0);
  const int *local = it.row_local + it.row_off[k] + r0;
  const int *perm = it.perm + it.pdof_off[k];
  for (int s = threadIdx.x; s < TPW * kLuWaves * kLuNb; s += kLuThreads) {
    const int c = min(max(perm[min(s, m - 1)], 0), m - 1);
    prow[s] = c;
    scale[s] = it.er ? it.er[it.dof[it.pdof_off[k] + c]] : 0;
  }
  T *W = it.W + it.woff[k] + (int64_t)r0 * m;
  __syncthreads();
  const int first = local[0];   // the rows are in ascending order
  for (int v0 = 0; v0 < nr; v0 += 16 * G) {
    int pos[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int r = v0 + 16 * g + jl;
      pos[g] = r < nr ? local[r] : -1;
    }
    typename MM::acc x[TPW][G];
    lu_rows<T, TPW, TPW, G>(
        it.blocks + it.boff[k], m, block_ld(m), prow, pos, min(G, (nr - v0 + 15) / 16), (v0 ? local[v0] : first) / kLuNb,
        [](int) { return 0; }, [&](int) { return m; }, bc, x);
#pragma unroll
    for (int u = 0; u < TPW; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = (wave + kLuWaves * u) * kLuNb + MM::row(r, kq);
        if (s < m) {
          const int c = prow[s], er = scale[s];
          float top = 0.f;
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const int i = v0 + 16 * g + jl;
            if (i < nr) {
              const T y = ldexp(x[u][g][r], er);
              W[(int64_t)c * nr + i] = y;
              top = fmaxf(top, fabsf((float)y));
            }
          }
          if (it.cscale) {
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
            if (jl == 0) atomicMax(reinterpret_cast<unsigned *>(it.cscale + it.pdof_off[k]) + c, __float_as_uint(top));
          }
        }
      }
    __syncthreads();
  }
}

// 16-bit copy of the rows that k_lu_rows left in FP32, one workgroup per
// task: row r is stored divided by the column scales and by its row scale,
// the largest |w| / cs[c] of the row, in the grouped layout (see
// launch_pack_owned), or without woff16 in the plain one.  Lane r of every
// wave holds row r, the waves share the columns; in the grouped layout four
// columns make one 8-byte store a lane.
template <int KIND>
__global__ __launch_bounds__(256) void k_pack16_rows(const float *__restrict__ rows, const int *__restrict__ pm,
                                                     const int *__restrict__ po, const int *__restrict__ row_off,
                                                     const int64_t *__restrict__ pdof_off,
                                                     const int64_t *__restrict__ woff,
                                                     const int64_t *__restrict__ woff16,
                                                     const int *__restrict__ task_patch,
                                                     const int *__restrict__ task_row0,
                                                     const float *__restrict__ cscale, uint16_t *__restrict__ W16,
                                                     float *__restrict__ wscale) {
  __shared__ double part[4][64];
  const int k = task_patch[blockIdx.x], r0 = task_row0[blockIdx.x], m = pm[k];
  const int nr = min(64, po[k] - r0), r = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rc = min(r, nr - 1);
  const float *W = rows + woff[k] + (int64_t)r0 * m + rc, *cs = cscale + pdof_off[k];
  double top = 0.0;
#pragma unroll 8
  for (int c = wave; c < m; c += 4) top = fmax(top, fabs((double)W[c * nr]) / (double)cs[c]);
  part[wave][r] = top;
  __syncthreads();
  top = fmax(fmax(part[0][r], part[1][r]), fmax(part[2][r], part[3][r]));
  if (top == 0.0) top = 1.0;
  if (r >= nr) return;
  if (wave == 0) wscale[row_off[k] + r0 + r] = (float)top;
  auto rounded = [&](int c) -> uint16_t {
    if (c >= m) return 0;
    const float v = (float)((double)W[c * nr] / ((double)cs[c] * top));
    if constexpr (KIND == 1) {
      const __hip_bfloat16 b = __float2bfloat16(v);
      return *reinterpret_cast<const uint16_t *>(&b);
    } else {
      const __half b = __float2half(v);
      return *reinterpret_cast<const uint16_t *>(&b);
    }
  };
  if (!woff16) {
    uint16_t *out = W16 + woff[k] + (int64_t)r0 * m + r;
    for (int c = wave; c < m; c += 4) out[c * nr] = rounded(c);
    return;
  }
  const int m4 = (m + 3) & ~3;
  uint16_t *out = W16 + woff16[k] + (int64_t)r0 * m4 + 4 * r;
#pragma unroll 2
  for (int c = 4 * wave; c < m; c += 16) {
    ushort4 q;
    q.x = rounded(c), q.y = rounded(c + 1), q.z = rounded(c + 2), q.w = rounded(c + 3);
    *reinterpret_cast<ushort4 *>(out + (c / 4) * 4 * nr) = q;
  }
}

// The instance for blocks of up to mmax dofs, to f as its rows a lane of the
// factoring wave (registers for the largest block) and panel buffers (two of
// more than 512 FP64 rows do not fit in LDS).
template <typename T, class F>
static auto lu_blocks_class(int mmax, F f) {
  if (mmax <= 128) return f(std::integral_constant<int, 2>(), std::integral_constant<int, 2>());
  if (mmax <= 256) return f(std::integral_constant<int, 4>(), std::integral_constant<int, 2>());
  if (mmax <= 384) return f(std::integral_constant<int, 6>(), std::integral_constant<int, 2>());
  if (mmax <= 512) return f(std::integral_constant<int, 8>(), std::integral_constant<int, 2>());
  return f(std::integral_constant<int, 13>(), std::integral_constant<int, sizeof(T) == 8 ? 1 : 2>());
}
template <typename T>
hipError_t lu_blocks_prepare(int mmax) {
  return lu_blocks_class<T>(mmax, [](auto rmax, auto pb) {
    static std::atomic<uint64_t> devices{0};
    return allow_lds(devices, (const void *)k_lu_blocks<T, rmax(), pb()>,
                     lu_lds_bytes<T>(block_ld(std::min(64 * rmax(), kMaxPatch)), pb()));
  });
}
template hipError_t lu_blocks_prepare<double>(int);
template hipError_t lu_blocks_prepare<float>(int);
template <typename T>
void launch_lu_blocks(T *blocks, const int64_t *boff, const int *pm, const int64_t *poff, int *perm, int *status,
                      const int *order, int nblk, int mmax, hipStream_t st, hipEvent_t ev0) {
  if (nblk == 0) return;
  lu_blocks_class<T>(mmax, [&](auto rmax, auto pb) {
    hipExtLaunchKernelGGL((k_lu_blocks<T, rmax(), pb()>), dim3(nblk), dim3(kLuThreads),
                          lu_lds_bytes<T>(block_ld(mmax), pb()), st, ev0, nullptr, 0, blocks, boff, pm, poff, perm,
                          status, order);
  });
}
template void launch_lu_blocks<double>(double *, const int64_t *, const int *, const int64_t *, int *, int *,
                                       const int *, int, int, hipStream_t, hipEvent_t);
template void launch_lu_blocks<float>(float *, const int64_t *, const int *, const int64_t *, int *, int *,
                                      const int *, int, int, hipStream_t, hipEvent_t);

template <typename T>
void launch_lu_rows(const LuRowsItem<T> *items, const int *ntasks, int count, int mmax, hipStream_t st,
                    hipEvent_t ev1) {
  for (int i0 = 0; i0 < count; i0 += kLuRowsItems) {
    LuRowsBatch<T> B;
    B.count = std::min(count - i0, kLuRowsItems);
    B.task0[0] = 0;
    for (int i = 0; i < B.count; ++i) {
      B.it[i] = items[i0 + i];
      B.task0[i + 1] = B.task0[i] + ntasks[i0 + i];
    }
    const int ntask = B.task0[B.count], chunk = (ntask + 7) / 8;
    if (ntask == 0) continue;
    const hipEvent_t ev = i0 + kLuRowsItems >= count ? ev1 : nullptr;
#define FSI_LU_ROWS(TPW, G)                                                                                  \
  hipExtLaunchKernelGGL((k_lu_rows<T, TPW, G>), dim3(8 * chunk), dim3(kLuThreads), 0, st, nullptr, ev, 0, B, \
                        ntask, chunk)
    // panels a wave: registers for the largest block
    if (mmax <= 128)
      FSI_LU_ROWS(1, 4);
    else if (mmax <= 256)
      FSI_LU_ROWS(2, 4);
    else if (mmax <= 384)
      FSI_LU_ROWS(3, 4);
    else if (mmax <= 512)
      FSI_LU_ROWS(4, (sizeof(T) == 8 ? 2 : 4));
    else
      FSI_LU_ROWS(7, (sizeof(T) == 8 ? 2 : 4));
#undef FSI_LU_ROWS
  }
}
template void launch_lu_rows<double>(const LuRowsItem<double> *, const int *, int, int, hipStream_t, hipEvent_t);
template void launch_lu_rows<float>(const LuRowsItem<float> *, const int *, int, int, hipStream_t, hipEvent_t);

template <typename T>
void launch_scale_rows(const CsrView<double> &J, T *out, int *er, hipStream_t st) {
  if (J.nrows > 0) k_scale_rows<T><<<(J.nrows + 15) / 16, 256, 0, st>>>(J.nrows, J.rowptr, J.val, out, er);
}
template void launch_scale_rows<double>(const CsrView<double> &, double *, int *, hipStream_t);
template void launch_scale_rows<float>(const CsrView<double> &, float *, int *, hipStream_t);

void launch_pack16_rows(const float *rows, const int *pm, const int *po, const int *row_off, const int64_t *pdof_off,
                        const int64_t *woff, const int64_t *woff16, const int *task_patch, const int *task_row0,
                        int ntask, const float *cscale, uint16_t *W16, int w16_kind, float *wscale, hipStream_t st) {
  if (ntask == 0) return;
  if (w16_kind == 1)
    k_pack16_rows<1><<<ntask, 256, 0, st>>>(rows, pm, po, row_off, pdof_off, woff, woff16, task_patch, task_row0,
                                            cscale, W16, wscale);
  else
    k_pack16_rows<2><<<ntask, 256, 0, st>>>(rows, pm, po, row_off, pdof_off, woff, woff16, task_patch, task_row0,
                                            cscale, W16, wscale);
}

}  // namespace fsi
