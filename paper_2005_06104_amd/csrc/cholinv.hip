// Cholesky factorisation G = L L^H of a Hermitian positive definite n x n
// matrix (n <= 512, row-major complex128) together with L^-1, in one
// cooperative launch over the 16 x 16 blocks (i, k), k <= i, of the lower
// triangle (tiled right-looking order, each update applied as soon as its
// operands exist):
//     L_ik = (G_ik - sum_{j<k} L_ij L_kj^H) (L_kk^-1)^H           k < i,
//     L_ii = chol(G_ii - sum_{j<i} L_ij L_ij^H),  with L_ii^-1,
//     Linv_ik = -L_ii^-1 sum_{j=k}^{i-1} L_ij Linv_jk              k < i.
// The chain along the diagonal is what is sequential, and a block handed from
// one workgroup to another costs two to three microseconds (write back, flag,
// poll, fetch).  So one workgroup per matrix runs the whole chain out of LDS,
// the diagonal blocks and those below them: while two of its waves factorise
// and invert block (i, i), two others bring block row i + 1 up to date with
// L_{i+1,i-1}, and one writes out the step before.  The other blocks have a
// workgroup each; those of (i, i) and (i, i - 1) hand the chain their sums over
// j < i - 2, early enough for it not to wait.  n = 300: 160 us, 8.2 us a block row (each
// diagonal block in a workgroup of its own, LDS and shuffles: 335 us).
// A block is published with a flag once written; a workgroup waits only for
// blocks of lower column index (or, for L^-1, of lower row index in its own
// column) and for diagonal blocks, so the waits form chains that end.  Every
// wait is bounded; one that runs out makes the call report failure.  The
// factorisation reports failure when a pivot is not positive and finite.
// Block-diagonal matrices (the Gram matrices of charged tensors, whose
// charge sectors are contiguous) are factorised sector by sector in the same
// launch: each sector has its own workgroups and flags, and the blocks
// between sectors are never read.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "wave.h"

namespace {

constexpr int CB = 16;            // block size
constexpr int CNT = 256;          // threads of a block's workgroup
constexpr int CNTD = CNT + 64;    // of the diagonal chain's, and of the launch
constexpr int CMAXB = 32;         // block rows at most
constexpr int CENT = CB * CB / CNT;   // tile entries per thread
constexpr int CPR = CNT / CB;         // threads per tile row
constexpr int NPART = 64 / CB;        // lanes per row in the one-wave steps
static_assert(CENT >= 1 && CB * CB == CENT * CNT && CB == 16 && NPART == 4, "tile mapping");
constexpr int CFLAG = 16;         // one 64-byte line per flag
constexpr unsigned CSPIN = 1u << 22;
constexpr int CMAXSEC = 64;       // sectors per launch
constexpr int CMAXWG = 768;       // workgroups per launch (all co-resident: three of five waves on each of 256 CUs)
constexpr size_t CSEC_FLAGS = 2 * CMAXB * CMAXB * CFLAG;   // flag words per sector

struct CholArgs {
  const double2* G;   // ld x ld, Hermitian (the lower blocks of each sector are read)
  double2* L;         // out: the lower blocks of L in each sector (may be G)
  double2* Li;        // out: L^-1 in each sector (zero above the diagonal)
  unsigned* flags;    // CSEC_FLAGS per sector, zero at launch
  int* info;          // 0 at launch; 1 not positive definite, 2 a wait ran out
  int ld, nsec;
  int off[CMAXSEC], size[CMAXSEC], wg0[CMAXSEC + 1];   // sector s: rows off..off+size, workgroups wg0[s]..
};

// one sector as the workgroup sees it
struct Sec {
  const double2* G;
  double2* L;
  double2* Li;
  unsigned* fl;       // block (i, k) of L published (k = i: with L_ii^-1)
  unsigned* fi;       // block (i, k) of L^-1 published (i > k)
  int* info;
  int n, ld;
};

__device__ inline double2 cm(double2 a, double2 b) { return double2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ inline double2 cmc(double2 a, double2 b) {   // a * conj(b)
  return double2{a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y};
}

__device__ inline int bsize(const Sec& a, int i) { return min(CB, a.n - i * CB); }

__device__ inline unsigned* flag_at(unsigned* f, int r, int c) { return f + (r * CMAXB + c) * CFLAG; }

// wait until the flags f1 and f2 are set; false when a wait ran out or
// another workgroup gave up
__device__ bool wait_flags(const Sec& a, const unsigned* f1, const unsigned* f2, int* s_ok) {
  if (threadIdx.x == 0) {
    unsigned polls = 0;
    int ok = 1;
    while (__hip_atomic_load(f1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u ||
           __hip_atomic_load(f2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
      if (__hip_atomic_load(a.info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2 || ++polls > CSPIN) {
        __hip_atomic_store(a.info, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *s_ok = ok;
  }
  __syncthreads();
  return *s_ok != 0;
}

// set flag f once the workgroup's stores before the call are done
__device__ void publish(unsigned* f) {
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(f, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// tile[r][c] = M[(r0 + r) * n + c0 + c] for r < rows, c < cols; zero elsewhere
__device__ void load_tile(double2 (*t)[CB + 1], const double2* M, int n, int r0, int rows, int c0, int cols) {
  for (int e = threadIdx.x; e < CB * CB; e += CNT) {
    const int r = e / CB, c = e % CB;
    t[r][c] = (r < rows && c < cols) ? M[(size_t)(r0 + r) * n + c0 + c] : double2{0.0, 0.0};
  }
}

__device__ void store_tile(const double2 (*t)[CB + 1], double2* M, int n, int r0, int rows, int c0, int cols) {
  for (int e = threadIdx.x; e < CB * CB; e += CNT) {
    const int r = e / CB, c = e % CB;
    if (r < rows && c < cols) M[(size_t)(r0 + r) * n + c0 + c] = t[r][c];
  }
}

// acc[q] (the thread's entries of a tile: row tid / CPR, columns
// (tid % CPR) + CPR q) += sign * (X Y^H) or sign * (X Y)
template <bool HERM>
__device__ void tile_mma(double2 acc[CENT], const double2 (*X)[CB + 1], const double2 (*Y)[CB + 1], double sign) {
  const int r = threadIdx.x / CPR, c0 = threadIdx.x % CPR;
#pragma unroll 4
  for (int k = 0; k < CB; ++k) {
    const double2 x = X[r][k];
#pragma unroll
    for (int q = 0; q < CENT; ++q) {
      const int c = c0 + CPR * q;
      const double2 p = HERM ? cmc(x, Y[c][k]) : cm(x, Y[k][c]);
      acc[q].x += sign * p.x;
      acc[q].y += sign * p.y;
    }
  }
}

__device__ void acc_to_tile(const double2 acc[CENT], double2 (*t)[CB + 1]) {
  const int r = threadIdx.x / CPR, c0 = threadIdx.x % CPR;
#pragma unroll
  for (int q = 0; q < CENT; ++q) t[r][c0 + CPR * q] = acc[q];
}

__device__ void tile_to_acc(const double2 (*t)[CB + 1], double2 acc[CENT]) {
  const int r = threadIdx.x / CPR, c0 = threadIdx.x % CPR;
#pragma unroll
  for (int q = 0; q < CENT; ++q) acc[q] = t[r][c0 + CPR * q];
}

// The mi x mi diagonal block in tS (the lower part; the strict upper part holds
// the matrix) is factorised in place by one wave; *s_fail becomes 1 when a pivot
// is not positive and finite.  Left-looking, row rr on the NPART lanes rr + CB p,
// each with the columns k = p mod NPART in registers: column c of L from the dot
// products of the rows with row c (broadcast within the row of lanes), every
// lane adding its NPART-th of the terms.  Another wave forms the inverse in tY a
// row behind by forward substitution, column j on the lanes j + CB p; the first
// tells it in *done how many columns are there (a wave's LDS accesses keep their
// order).  A wave issues an instruction every four to five cycles, and the two
// are about 80 each per column: in one wave they took 8.7 us a block, in two
// 6.1.  FULL: mi = CB, the usual case, without the bounds.
struct DiagShare {
  double il[CB];   // 1 / L[c][c]
  int done;        // columns of L that are in tS; 0 at the start
};
template <int C>
__device__ inline void diag_column(double2 (*tS)[CB + 1], DiagShare* sh, double2 (&lr)[CB / NPART], int& bad, int rr,
                                   int part) {
  const double2 v = tS[rr][C];
  double2 t{0.0, 0.0};
#pragma unroll
  for (int m = 0; NPART * m < C; ++m) {
    const double2 lc{wave::row_bcast<C>(lr[m].x), wave::row_bcast<C>(lr[m].y)};
    t.x += fma(lr[m].x, lc.x, lr[m].y * lc.y);   // zero where k >= C
    t.y += fma(lr[m].y, lc.x, -(lr[m].x * lc.y));
  }
  t.x = wave::rows_sum(t.x);
  t.y = wave::rows_sum(t.y);
  const double d = wave::row_bcast<C>(v.x - t.x);
  const bool good = d > 0.0 && isfinite(d);
  bad |= good ? 0 : 1;
  const double l = good ? sqrt(d) : 1.0, il = 1.0 / l;
  double2 x{(v.x - t.x) * il, (v.y - t.y) * il};
  if (rr == C) x = double2{l, 0.0};
  if (rr < C) x = double2{0.0, 0.0};
  if (part == C % NPART) {
    lr[C / NPART] = x;   // L[rr][p + NPART m]
    tS[rr][C] = x;
  }
  asm volatile("" ::: "memory");
  if (rr == 0 && part == 0) {
    sh->il[C] = il;
    asm volatile("" ::: "memory");
    __hip_atomic_store(&sh->done, C + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  asm volatile("" ::: "memory");
}
template <bool FULL, int C>
__device__ inline void diag_columns(double2 (*tS)[CB + 1], DiagShare* sh, double2 (&lr)[CB / NPART], int& bad, int mi,
                                    int rr, int part) {
  if constexpr (C < CB) {
    if (FULL || C < mi) diag_column<C>(tS, sh, lr, bad, rr, part);
    diag_columns<FULL, C + 1>(tS, sh, lr, bad, mi, rr, part);
  }
}
// row R of L^-1: x_R (column j < R) = -(sum_{q=j}^{R-1} L[R][q] x_q) / L[R][R]
template <bool FULL, int R>
__device__ inline void diag_inverse_rows(const double2 (*tS)[CB + 1], double2 (*tY)[CB + 1], DiagShare* sh,
                                         double2 (&y)[CB / NPART], unsigned& polls, int mi, int j, int part) {
  if constexpr (R < CB) {
    if (FULL || R < mi) {
      // the factor's wave always gets there, bad pivots or not; bounded all the same
      while (__hip_atomic_load(&sh->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= R && polls <= CSPIN)
        ++polls;
      asm volatile("" ::: "memory");
      double2 t{0.0, 0.0};
#pragma unroll
      for (int m = 0; NPART * m < R; ++m) {
        const int q = j + part + NPART * m;
        const double2 l = tS[R][q < CB ? q : CB - 1];
        const double px = fma(l.x, y[m].x, -(l.y * y[m].y)), py = fma(l.y, y[m].x, l.x * y[m].y);
        t.x += q < R ? px : 0.0;
        t.y += q < R ? py : 0.0;
      }
      t.x = wave::rows_sum(t.x);
      t.y = wave::rows_sum(t.y);
      const double ir = sh->il[R];
      double2 x{-t.x * ir, -t.y * ir};
      if (j == R) x = double2{ir, 0.0};
      if (j > R) x = double2{0.0, 0.0};
#pragma unroll
      for (int m = 0; m < CB / NPART; ++m)
        if (R - j - part == NPART * m) y[m] = x;   // L^-1[j + p + NPART m][j]
      if (part == 0) tY[R][j] = x;
    }
    diag_inverse_rows<FULL, R + 1>(tS, tY, sh, y, polls, mi, j, part);
  }
}
// entries past the block
__device__ inline void diag_clear(double2 (*t)[CB + 1], int mi, int lane) {
  for (int e = lane; e < CB * CB; e += 64)
    if (e / CB >= mi || e % CB >= mi) t[e / CB][e % CB] = double2{0.0, 0.0};
  asm volatile("" ::: "memory");
}
__device__ void diag_factor(double2 (*tS)[CB + 1], int mi, DiagShare* sh, int* s_fail, int lane) {
  double2 lr[CB / NPART];
#pragma unroll
  for (int m = 0; m < CB / NPART; ++m) lr[m] = double2{0.0, 0.0};
  int bad = 0;
  if (mi == CB) {
    diag_columns<true, 0>(tS, sh, lr, bad, mi, lane % CB, lane / CB);
  } else {
    diag_clear(tS, mi, lane);
    diag_columns<false, 0>(tS, sh, lr, bad, mi, lane % CB, lane / CB);
  }
  if (lane == 0) *s_fail = bad;
}
// false when the wait for the factor ran out
__device__ bool diag_invert(const double2 (*tS)[CB + 1], double2 (*tY)[CB + 1], int mi, DiagShare* sh, int lane) {
  double2 y[CB / NPART];
#pragma unroll
  for (int m = 0; m < CB / NPART; ++m) y[m] = double2{0.0, 0.0};
  unsigned polls = 0;
  if (mi == CB) {
    diag_inverse_rows<true, 0>(tS, tY, sh, y, polls, mi, lane % CB, lane / CB);
  } else {
    diag_clear(tY, mi, lane);
    diag_inverse_rows<false, 0>(tS, tY, sh, y, polls, mi, lane % CB, lane / CB);
  }
  return polls <= CSPIN;
}

// workgroup barrier for LDS alone: stores to memory stay in flight
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The steps of single waves.  Lane l holds the entries e = l + 64 q of a tile.
constexpr int WENT = CB * CB / 64;

// wait_flags for one wave and one flag
__device__ bool wave_wait(const Sec& a, const unsigned* f) {
  unsigned polls = 0;
  while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
    if (__hip_atomic_load(a.info, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2 || ++polls > CSPIN) {
      __hip_atomic_store(a.info, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return true;
}
__device__ void wave_load(double2 (&v)[WENT], const double2* M, int ld, int r0, int rows, int c0, int cols, int lane) {
#pragma unroll
  for (int q = 0; q < WENT; ++q) {
    const int r = (lane + 64 * q) / CB, c = lane % CB;
    v[q] = (r < rows && c < cols) ? M[(size_t)(r0 + r) * ld + c0 + c] : double2{0.0, 0.0};
  }
}
__device__ void wave_store(const double2 (*t)[CB + 1], double2* M, int ld, int r0, int rows, int c0, int cols,
                           int lane) {
#pragma unroll
  for (int q = 0; q < WENT; ++q) {
    const int r = (lane + 64 * q) / CB, c = lane % CB;
    if (r < rows && c < cols) M[(size_t)(r0 + r) * ld + c0 + c] = t[r][c];
  }
}
__device__ void wave_to_tile(const double2 (&v)[WENT], double2 (*t)[CB + 1], int lane) {
#pragma unroll
  for (int q = 0; q < WENT; ++q) t[(lane + 64 * q) / CB][lane % CB] = v[q];
}
// v -= X Y^H
__device__ void wave_sub(double2 (&v)[WENT], const double2 (*X)[CB + 1], const double2 (*Y)[CB + 1], int lane) {
#pragma unroll 4
  for (int k = 0; k < CB; ++k)
#pragma unroll
    for (int q = 0; q < WENT; ++q) {
      const double2 p = cmc(X[(lane + 64 * q) / CB][k], Y[lane % CB][k]);
      v[q].x += -1.0 * p.x;
      v[q].y += -1.0 * p.y;
    }
}

struct ChainTiles {
  double2 (*S)[CB + 1];    // the diagonal block, then its factor
  double2 (*Y)[CB + 1];    // the factor's inverse
  double2 (*C)[CB + 1];    // L_{i+1,i}
  double2 (*A)[CB + 1];    // block (i + 1, i), up to date but for column i
  double2 (*B)[CB + 1];    // block (i + 1, i + 1), up to date but for column i
  double2 (*X1)[CB + 1];   // L_{i+1,i-1}, one copy per wave that uses it
  double2 (*X2)[CB + 1];
};

// The chain along the diagonal of one matrix, all CNTD threads.
__device__ void diagonal_chain(const Sec& a, const ChainTiles& t, DiagShare* sh, int* s_ok, int* s_fail) {
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int nb = (a.n + CB - 1) / CB, ld = a.ld;
  if (tid == 0) {
    *s_ok = 1;
    *s_fail = 0;
    sh->done = 0;
  }
  if (tid < CNT) load_tile(t.S, a.G, ld, 0, bsize(a, 0), 0, bsize(a, 0));
  lds_barrier();
  for (int i = 0; i < nb; ++i) {
    const int r = i + 1, mi = bsize(a, i), ri = i * CB, rr = r * CB;
    const bool more = r < nb;
    const int mr = more ? bsize(a, r) : 0;
    if (wave == 0) {
      diag_factor(t.S, mi, sh, s_fail, lane);
    } else if (wave == 3) {
      if (!diag_invert(t.S, t.Y, mi, sh, lane) && lane == 0) {
        __hip_atomic_store(a.info, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_ok = 0;
      }
    } else if ((wave == 1 || wave == 2) && more) {
      // wave 1: block (r, i), wave 2: block (r, r), from their workgroups' sums
      // over j < r - 2 (none for r < 3), with column j = i - 1 added here
      const bool dia = wave == 2;
      const double2 (*x)[CB + 1] = dia ? t.X2 : t.X1;
      bool ok = r < 3 || wave_wait(a, dia ? flag_at(a.fi, r, r) : flag_at(a.fl, i, r));
      if (ok) {
        double2 v[WENT];
        wave_load(v, r < 3 ? a.G : a.L, ld, rr, mr, dia ? rr : ri, dia ? mr : mi, lane);
        if (i >= 1) {
          ok = wave_wait(a, flag_at(a.fl, r, i - 1));
          if (ok) {
            double2 xv[WENT];
            wave_load(xv, a.L, ld, rr, mr, ri - CB, CB, lane);
            wave_to_tile(xv, dia ? t.X2 : t.X1, lane);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            wave_sub(v, x, dia ? x : t.C, lane);
          }
        }
        wave_to_tile(v, dia ? t.B : t.A, lane);
      }
      if (!ok && lane == 0) *s_ok = 0;
    } else if (wave == 4 && i > 0) {
      // this wave wrote the blocks of the step before
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (lane == 0) {
        __hip_atomic_store(flag_at(a.fl, i - 1, i - 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(flag_at(a.fl, i, i - 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    lds_barrier();
    if (*s_ok == 0) return;
    if (tid == 0) sh->done = 0;
    if (tid == 0 && *s_fail) __hip_atomic_store(a.info, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // L_ri = A (L_ii^-1)^H
    if (wave == 4) {
      wave_store(t.S, a.L, ld, ri, mi, ri, mi, lane);
      wave_store(t.Y, a.Li, ld, ri, mi, ri, mi, lane);
    } else if (more) {
      double2 acc[CENT];
#pragma unroll
      for (int q = 0; q < CENT; ++q) acc[q] = double2{0.0, 0.0};
      tile_mma<true>(acc, t.A, t.Y, 1.0);
      acc_to_tile(acc, t.C);
    }
    lds_barrier();
    // the next diagonal block: B - L_ri L_ri^H
    if (more) {
      if (wave == 4) {
        wave_store(t.C, a.L, ld, rr, mr, ri, mi, lane);
      } else {
        double2 acc[CENT];
        tile_to_acc(t.B, acc);
        tile_mma<true>(acc, t.C, t.C, -1.0);
        acc_to_tile(acc, t.S);
      }
    }
    lds_barrier();
  }
  if (wave == 4) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane == 0)
      __hip_atomic_store(flag_at(a.fl, nb - 1, nb - 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__global__ __launch_bounds__(CNTD, 4) void cholinv_kernel(CholArgs args) {
  __shared__ double2 tS[CB][CB + 1], tX[CB][CB + 1], tY[CB][CB + 1];
  __shared__ double2 tA[CB][CB + 1], tB[CB][CB + 1], tC[CB][CB + 1], tX2[CB][CB + 1];
  __shared__ DiagShare diag;
  __shared__ int s_ok, s_fail;
  int sec = 0;
  while (sec + 1 < args.nsec && args.wg0[sec + 1] <= (int)blockIdx.x) ++sec;
  const int wg = (int)blockIdx.x - args.wg0[sec];
  Sec a;
  {
    const size_t o = (size_t)args.off[sec] * args.ld + args.off[sec];
    a.G = args.G + o;
    a.L = args.L + o;
    a.Li = args.Li + o;
    a.fl = args.flags + sec * CSEC_FLAGS;
    a.fi = a.fl + CMAXB * CMAXB * CFLAG;
    a.info = args.info;
    a.n = args.size[sec];
    a.ld = args.ld;
  }
  if (wg == 0) {   // block (0, 0) and the chain
    const ChainTiles t{tS, tY, tC, tA, tB, tX, tX2};
    diagonal_chain(a, t, &diag, &s_ok, &s_fail);
    return;
  }
  if (threadIdx.x >= CNT) return;
  int i = 0;
  while ((i + 1) * (i + 2) / 2 <= wg) ++i;
  const int k = wg - i * (i + 1) / 2;
  const int n = a.ld, mi = bsize(a, i), mk = bsize(a, k), ri = i * CB, rk = k * CB;
  double2 acc[CENT];

  // ---- S = G_ik - sum_j L_ij L_kj^H over j < k (blocks j < k are full), for
  // the blocks of the chain over j < i - 2
  const bool chain = k + 1 >= i;
  const int jn = chain ? i - 2 : k;
  if (!chain || jn > 0) {
    load_tile(tS, a.G, n, ri, mi, rk, mk);
    __syncthreads();
    tile_to_acc(tS, acc);
    for (int j = 0; j < jn; ++j) {
      if (!wait_flags(a, flag_at(a.fl, i, j), flag_at(a.fl, k, j), &s_ok)) return;
      load_tile(tX, a.L, n, ri, mi, j * CB, CB);                     // L_ij
      if (i != k) load_tile(tY, a.L, n, rk, mk, j * CB, CB);         // L_kj
      __syncthreads();
      tile_mma<true>(acc, tX, i == k ? tX : tY, -1.0);
      __syncthreads();
    }
  }
  if (chain) {
    if (jn > 0) {   // handed over in the block's place in L
      acc_to_tile(acc, tS);
      __syncthreads();
      store_tile(tS, a.L, n, ri, mi, rk, mk);
      publish(i == k ? flag_at(a.fi, i, i) : flag_at(a.fl, k, i));
    }
    if (i == k) return;
    if (!wait_flags(a, flag_at(a.fl, i, k), flag_at(a.fl, k, k), &s_ok)) return;
    load_tile(tX, a.L, n, ri, mi, rk, mk);
    load_tile(tY, a.Li, n, rk, mk, rk, mk);
    __syncthreads();
  } else {
    // ---- L_ik = S (L_kk^-1)^H, kept in tX
    if (!wait_flags(a, flag_at(a.fl, k, k), flag_at(a.fl, k, k), &s_ok)) return;
    acc_to_tile(acc, tS);
    load_tile(tY, a.Li, n, rk, mk, rk, mk);                          // L_kk^-1
    __syncthreads();
    for (int q = 0; q < CENT; ++q) acc[q] = double2{0.0, 0.0};
    tile_mma<true>(acc, tS, tY, 1.0);
    acc_to_tile(acc, tX);
    __syncthreads();
    store_tile(tX, a.L, n, ri, mi, rk, mk);
    publish(flag_at(a.fl, i, k));
  }
  for (int e = threadIdx.x; e < CB * CB; e += CNT) {                   // block (k, i) of L^-1
    const int y = e / CB, x = e % CB;
    if (y < mk && x < mi) a.Li[(size_t)(rk + y) * n + ri + x] = double2{0.0, 0.0};
  }

  // ---- Linv_ik = -L_ii^-1 sum_{j=k}^{i-1} L_ij Linv_jk (blocks j < i are full)
  for (int q = 0; q < CENT; ++q) acc[q] = double2{0.0, 0.0};
  tile_mma<false>(acc, tX, tY, 1.0);                                 // j = k: L_ik L_kk^-1
  __syncthreads();
  for (int j = k + 1; j < i; ++j) {
    if (!wait_flags(a, flag_at(a.fl, i, j), flag_at(a.fi, j, k), &s_ok)) return;
    load_tile(tX, a.L, n, ri, mi, j * CB, CB);                       // L_ij
    load_tile(tY, a.Li, n, j * CB, CB, rk, mk);                      // Linv_jk
    __syncthreads();
    tile_mma<false>(acc, tX, tY, 1.0);
    __syncthreads();
  }
  if (!wait_flags(a, flag_at(a.fl, i, i), flag_at(a.fl, i, i), &s_ok)) return;
  acc_to_tile(acc, tS);
  load_tile(tX, a.Li, n, ri, mi, ri, mi);                            // L_ii^-1
  __syncthreads();
  for (int q = 0; q < CENT; ++q) acc[q] = double2{0.0, 0.0};
  tile_mma<false>(acc, tX, tS, -1.0);
  acc_to_tile(acc, tY);
  __syncthreads();
  store_tile(tY, a.Li, n, ri, mi, rk, mk);
  publish(flag_at(a.fi, i, k));
}

__global__ void cholinv_reset_kernel(unsigned* flags, int nf, int* info) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nf) flags[t] = 0u;
  if (t == 0 && info) *info = 0;
}

}  // namespace

namespace kern {

int cholinv_max_n() { return CB * CMAXB; }

size_t cholinv_scratch_bytes() { return sizeof(unsigned) * CSEC_FLAGS + 256; }

size_t cholinv_blocks_scratch_bytes() { return sizeof(unsigned) * CSEC_FLAGS * CMAXSEC + 256; }

hipError_t cholinv(hipStream_t s, const void* G, int n, void* L, void* Linv, int* info, void* scratch) {
  const int off = 0;
  return cholinv_blocks(s, G, n, &off, &n, 1, L, Linv, info, scratch, false);
}

hipError_t cholinv_blocks(hipStream_t s, const void* G, int ld, const int* off, const int* size, int nsec, void* L,
                          void* Linv, int* info, void* scratch, bool keep_info) {
  if (ld < 1 || nsec < 1 || !scratch || !info) return hipErrorInvalidValue;
  for (int q = 0; q < nsec; ++q)
    if (size[q] < 1 || size[q] > CB * CMAXB || off[q] < 0 || off[q] + size[q] > ld) return hipErrorInvalidValue;
  // sectors go to launches of at most CMAXSEC sectors and CMAXWG workgroups
  bool first = true;
  for (int q0 = 0; q0 < nsec;) {
    CholArgs a{};
    a.G = static_cast<const double2*>(G);
    a.L = static_cast<double2*>(L);
    a.Li = static_cast<double2*>(Linv);
    a.flags = static_cast<unsigned*>(scratch);
    a.info = info;
    a.ld = ld;
    int wg = 0, q = q0;
    while (q < nsec && a.nsec < CMAXSEC) {
      const int nb = (size[q] + CB - 1) / CB, w = nb * (nb + 1) / 2;
      if (a.nsec > 0 && wg + w > CMAXWG) break;
      a.off[a.nsec] = off[q];
      a.size[a.nsec] = size[q];
      a.wg0[a.nsec] = wg;
      wg += w;
      ++a.nsec;
      ++q;
    }
    a.wg0[a.nsec] = wg;
    // flags of the sectors used; info once per call (a failure in an earlier
    // launch stays reported) unless the caller cleared it
    const int nf = (int)(CSEC_FLAGS * a.nsec);
    hipLaunchKernelGGL(cholinv_reset_kernel, dim3((nf + 255) / 256), dim3(256), 0, s, a.flags, nf,
                       first && !keep_info ? a.info : nullptr);
    void* args[] = {&a};
    const hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(cholinv_kernel), dim3(wg),
                                                    dim3(CNTD), args, 0, s);
    if (e != hipSuccess) return e;
    first = false;
    q0 = q;
  }
  return hipSuccess;
}

}  // namespace kern
