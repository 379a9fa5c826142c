// Device kernels of the GSE-TDVP1 hot path (gfx950 / CDNA4).
//
// * FP64 GEMM: a complex product as three real MFMA accumulations
//   (v_mfma_f64_16x16x4f64), the operands loaded straight in the MFMA layout.
// * complex64 GEMM: every operand as one, two or three BF16 terms on the BF16
//   matrix cores, which are sixteen times as fast as the FP32 ones; three
//   terms hold an FP32 number exactly.
//   These carry every contraction of the method: effective Hamiltonians,
//   environments, MPO application, basis extension.
// * wapply: contraction with the sparse MPO tensor over (MPO index, physical
//   index); memory bound.
// * complex128 vector helpers for the Lanczos recurrence (FP64 always).
#include <hip/hip_runtime.h>

#include <numeric>
#include <type_traits>

#include "common.h"
#include "wave.h"

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T> struct VT;
template <> struct VT<double> { using c2 = double2; };
template <> struct VT<float> { using c2 = float2; };

__device__ inline d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------- GEMM
// Block-sparse maps are built on output tiles of BM x BN.
constexpr int BM = 64, BN = 64;

// TAG only separates instantiations (the one-site effective Hamiltonian uses
// its own so that profilers and timers see it apart from the other GEMMs).
// Split-K: blockIdx.z = batch * S + split; split s covers k in
// [s*Kc, min(K, (s+1)*Kc)) and writes its partial product at C + s*sps.
// Block-sparse products (operands with U(1) charges): a linear grid over
// the work items kit (kern::KMap): item {tile, part, a, b} is output tile
// `tile` (batch entry outer) over the K intervals kiv[a .. b) as [x, y)
// pairs, its partial product at C + part * sps.  kit null: the dense tile
// grid over the whole K range (or one split-K part).  A tile with no
// interval writes alpha * 0 + beta * C.

// Operands are read by buffer loads at a uniform base and 32-bit offsets; an
// entry that is not there (past the operand, the sub-block or the interval)
// takes an offset past the buffer's 2^31 bytes and loads zero.
constexpr unsigned BUF_BYTES = 0x80000000u;

struct KIter {
  const int2* iv;
  int n;
  int2 one;
  __device__ int2 at(int v) const { return iv ? iv[v] : one; }
};

// the output tile, batch entry, split part and K range of this workgroup,
// and the rows r0 .. r1, columns c0 .. c1 of the tile it computes
struct TileJob {
  int m0, n0, split;
  int r0, r1, c0, c1;
  long long bz;
  KIter kr;
};

template <int TM, int TN>
__device__ inline TileJob tile_job(int M, int N, int K, int S, int Kc, const int4* __restrict__ kit,
                                   const int2* __restrict__ kiv) {
  TileJob j;
  const unsigned gx = gridDim.x, gy = gridDim.y, gz = gridDim.z;
  const unsigned lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  if (kit) {
    // items in decreasing K length: dispatch order (and the XCD round robin
    // of consecutive workgroups) spreads the long ones
    const int4 it = kit[2 * (size_t)lin], rg = kit[2 * (size_t)lin + 1];
    const int gxt = (N + BN - 1) / BN, tpb = gxt * ((M + BM - 1) / BM);
    j.bz = it.x / tpb;
    const int trem = it.x % tpb;
    j.m0 = (trem / gxt) * BM;
    j.n0 = (trem % gxt) * BN;
    j.split = it.y;
    j.r0 = rg.x;
    j.r1 = rg.y;
    j.c0 = rg.z;
    j.c1 = rg.w;
    j.kr.iv = kiv + it.z;
    j.kr.n = it.w - it.z;
    j.kr.one = make_int2(0, 0);
    return j;
  }
  // XCD-aware tile order: workgroups are dealt round-robin to the 8 XCDs, so
  // linear id g runs on XCD g % 8.  Give each XCD a contiguous band of tiles
  // (z-slice, then tile row, then tile column) so that the operand panels a
  // band needs stay in that XCD's L2.
  const unsigned tot = gx * gy * gz;
  const unsigned t = (tot % 8u == 0u) ? (lin % 8u) * (tot / 8u) + lin / 8u : lin;
  const unsigned tz = t / (gx * gy), trem = t % (gx * gy);
  j.m0 = (int)(trem / gx) * TM;
  j.n0 = (int)(trem % gx) * TN;
  j.bz = tz / S;
  j.split = tz % S;
  j.r0 = 0;
  j.r1 = TM;
  j.c0 = 0;
  j.c1 = TN;
  const int kb = j.split * Kc, ke = min(K, kb + Kc);
  j.kr.iv = nullptr;
  j.kr.n = kb < ke ? 1 : 0;
  j.kr.one = make_int2(kb, ke);
  return j;
}

// The wave's pieces of a block-sparse item: the product of ni rows and nj
// columns of 16 x 16 pieces at the tile offsets ro, co (on entry its quadrant
// of the 64 x 64 tile).  By quadrant, a sub-block covering part of the tile
// can leave some waves with four pieces and others with none, and the item
// lasts as long as its busiest wave.  An item whose covered pieces number at
// most four gets one per wave, one at most two pieces wide a row strip per
// wave, one at most two pieces tall a column strip per wave; larger ones keep
// the covered pieces of the quadrants.
__device__ inline void deal_pieces(const TileJob& job, bool mapped, int wave, int (&ro)[2], int (&co)[2], int& ni,
                                   int& nj) {
  if (!mapped) return;
  const int pi0 = job.r0 >> 4, pj0 = job.c0 >> 4;
  const int mi = ((job.r1 + 15) >> 4) - pi0, mj = ((job.c1 + 15) >> 4) - pj0;
  if (mi * mj <= 4) {   // one piece per wave
    ni = nj = wave < mi * mj ? 1 : 0;
    ro[0] = (pi0 + wave / mj) * 16;
    co[0] = (pj0 + wave % mj) * 16;
  } else if (mj <= 2) {   // row strips
    ni = wave < mi ? 1 : 0;
    nj = mj;
    ro[0] = (pi0 + wave) * 16;
    co[0] = pj0 * 16;
  } else if (mi <= 2) {   // column strips
    ni = mi;
    nj = wave < mj ? 1 : 0;
    ro[0] = pi0 * 16;
    co[0] = (pj0 + wave) * 16;
  } else {   // the covered part of the quadrant
    const int i0 = max(ro[0] >> 4, pi0), i1 = min((ro[0] >> 4) + 2, pi0 + mi);
    const int j0 = max(co[0] >> 4, pj0), j1 = min((co[0] >> 4) + 2, pj0 + mj);
    ni = max(i1 - i0, 0);
    nj = max(j1 - j0, 0);
    ro[0] = i0 * 16;
    co[0] = j0 * 16;
  }
  if (ni == 0 || nj == 0) ni = nj = ro[0] = co[0] = 0;
  ro[1] = ni == 2 ? ro[0] + 16 : ro[0];
  co[1] = nj == 2 ? co[0] + 16 : co[0];
}

// ---------------------------------------------------------------- BF16-term GEMM
// Complex GEMM on complex64 operands through the BF16 matrix cores with FP32
// accumulation (v_mfma_f32_16x16x32_bf16: lane l holds row l%16 and the eight
// k values 8*(l/16)..+7 of its operand; outputs as the f32 MFMA).  Each real
// number is written as a sum of TERMS BF16 numbers, each the nearest to what
// the ones before leave, and the products of two numbers whose terms' places
// add up to less than TERMS are formed, the smallest first:
//   TERMS 1: plain BF16 inputs;
//   TERMS 2: x = h + l, three products (about 16 bits);
//   TERMS 3: x = h + m + l exactly (24 bits), six products; what is left out
//            (m l, l m, l l) is less than 2^-24 of the product: |m| is at most
//            2^-8 / (1 + 2^-8) of x, |l| 2^-17 (x = 1 + 2^-8 - 2^-17: 2^-24.01).
// BF16 ends at 2^-133, FP32 at 2^-149: for TERMS 3 both operands are multiplied
// by 2^20 on the way in (exact) and the sums by 2^-40 on the way out, so that
// the last term of every normal FP32 number is there (2% of a large product's
// time).  What overflows on the way is formed again, see the store.
//
// What bounds it (TERMS 3, 20480 x 2048 x 1024): the matrix cores and the
// conversion at once; a K step of a 128 x 64 tile is 192 MFMAs a wave (3190
// cycles) and about 460 other vector instructions (2100), which the CU's two
// workgroups overlap in part: 1.86 ms, 184 TFLOP/s at 8 a complex
// multiply-add, 1.1 PFLOP/s in BF16 (a register-only loop of these MFMAs on
// such data: 1.9; a large library product in BF16: 1.2).  Both signs on A and
// in a step's sums, 64 more instructions: 1.93 ms.  The FP32 matrix cores in
// the 3M form: 2.67 ms.
constexpr int BKS = 32;
constexpr float UP3 = 0x1p20f;

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));

__device__ inline f4 mfma_bf16(uint4 a, uint4 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a), __builtin_bit_cast(bf8, b), c, 0, 0,
                                                  0);
}
// four k values a lane (v_mfma_f32_16x16x16_bf16: 4*(l/16)..+3)
__device__ inline f4 mfma_bf16(uint2 a, uint2 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4, a), __builtin_bit_cast(s4, b), c, 0, 0, 0);
}
__device__ inline uint2 bf16_flip(uint2 v, unsigned s) { return uint2{v.x ^ s, v.y ^ s}; }
__device__ inline uint4 bf16_flip(uint4 v, unsigned s) { return uint4{v.x ^ s, v.y ^ s, v.z ^ s, v.w ^ s}; }

// Operand tile of ROWS rows (m of A or n of B) x 32 k in chunks of eight
// consecutive k of one row, 4 ROWS / NTH of them per thread.  KC: k is the
// contiguous index in memory (the four chunks of a row on four neighbouring
// lanes, 64 bytes each); otherwise the rows are (neighbouring lanes on
// neighbouring rows, eight loads of eight bytes).
template <bool KC, int ROWS>
__device__ inline void chunk_at(int q, int& row, int& ch) {
  row = KC ? q >> 2 : q % ROWS;
  ch = KC ? q & 3 : q / ROWS;
}
// entry (row, chunk) of an LDS plane, k contiguous, 64 bytes a row: the chunks
// of a row are permuted by its place in the group of 16 so that neither the
// operand reads nor the stores of either order meet in a bank
__device__ inline int plane_at(int row, int ch) { return row * BKS + ((ch ^ (-(row >> 2) & 3)) << 3); }

// Chunk loads: the buffer's base is the tile's first row at k0, so a chunk
// costs one address register.  WIDE: leading dimensions whose tile reaches
// outside the buffer's 2^31 bytes, past its end or (negative ones) before its
// base, plain addresses.
constexpr long long LD_WIDE = 1LL << 20;   // 256 rows, 2^20 - 1 complex64 apart: just under 2^31 bytes
inline bool wide_ld(long long lda, long long ldb, long long limit) {
  return lda < 0 || ldb < 0 || lda >= limit || ldb >= limit;
}

template <bool KC, int ROWS, int NTH>
__device__ inline void chunk_offsets(long long ld, int r0, int R, int tid, unsigned (&off)[ROWS * 4 / NTH], int lo,
                                     int hi) {
#pragma unroll
  for (int it = 0; it < ROWS * 4 / NTH; ++it) {
    int row, ch;
    chunk_at<KC, ROWS>(tid + it * NTH, row, ch);
    const bool rok = r0 + row < R && row >= lo && row < hi;
    off[it] = rok ? (KC ? (unsigned)row * (unsigned)ld + 8u * ch : 8u * ch * (unsigned)ld + row) * 8u : BUF_BYTES;
  }
}

template <bool KC, bool WIDE, int ROWS, int NTH>
__device__ inline void chunk_load(const float2* __restrict__ X, long long ld, int r0, int R, int k0, int ke, int tid,
                                  const unsigned (&off)[ROWS * 4 / NTH], float2 (&v)[ROWS * 4 / NTH][8], int lo,
                                  int hi) {
  k0 = __builtin_amdgcn_readfirstlane(k0);   // uniform: the buffer's base is scalar
  ke = __builtin_amdgcn_readfirstlane(ke);
  if constexpr (WIDE) {
#pragma unroll
    for (int it = 0; it < ROWS * 4 / NTH; ++it) {
      int row, ch;
      chunk_at<KC, ROWS>(tid + it * NTH, row, ch);
      const int gr = r0 + row, gk = k0 + 8 * ch;
      const bool rok = gr < R && row >= lo && row < hi;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[it][j] = float2{0.f, 0.f};
        if (rok && gk + j < ke) v[it][j] = KC ? X[(long long)gr * ld + gk + j] : X[(long long)(gk + j) * ld + gr];
      }
    }
  } else {
    const float2* base = KC ? X + (long long)r0 * ld + k0 : X + (long long)k0 * ld + r0;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(base), 0, (int)BUF_BYTES, 0x00020000);
    const int ldb = (int)ld * 8;   // bytes from one k to the next (not KC)
    if (k0 + BKS <= ke) {
#pragma unroll
      for (int it = 0; it < ROWS * 4 / NTH; ++it) {
        unsigned o = off[it];
        asm("" : "+v"(o));   // one register and immediate offsets, not four sums kept through the loop
        if (KC) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const f4 w = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(o + 16u * j), 0, 0));
            v[it][2 * j] = float2{w.x, w.y};
            v[it][2 * j + 1] = float2{w.z, w.w};
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j)
            v[it][j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, j * ldb, 0));
        }
      }
    } else {   // the last step of an interval
#pragma unroll
      for (int it = 0; it < ROWS * 4 / NTH; ++it) {
        int row, ch;
        chunk_at<KC, ROWS>(tid + it * NTH, row, ch);
        const int left = ke - k0 - 8 * ch;
        unsigned o0 = off[it];
        asm("" : "+v"(o0));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const unsigned o = j < left ? o0 + (KC ? 8u * j : 0u) : BUF_BYTES;
          v[it][j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, KC ? 0 : j * ldb, 0));
        }
      }
    }
  }
}

// the TERMS BF16 terms of eight (uint4) or four (uint2) numbers (neg: of their
// negatives), packed
template <int TERMS, class V>
__device__ inline void bf16_terms(const float (&x)[sizeof(V) / 2], bool neg, V (&o)[TERMS]) {
  const float up = neg ? -UP3 : UP3;
  const unsigned flip = neg ? 0x80008000u : 0u;
  constexpr int P = sizeof(V) / 4;
  unsigned w[TERMS][P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    f2v v;
    v.x = TERMS == 3 ? x[2 * p] * up : x[2 * p];
    v.y = TERMS == 3 ? x[2 * p + 1] * up : x[2 * p + 1];
#pragma unroll
    for (int t = 0; t < TERMS; ++t) {
      w[t][p] = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf2));
      if (t + 1 < TERMS) {   // the rest, exact
        v.x -= __uint_as_float(w[t][p] << 16);
        v.y -= __uint_as_float(w[t][p] & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < TERMS; ++t) {
    if constexpr (P == 4) o[t] = uint4{w[t][0], w[t][1], w[t][2], w[t][3]};
    else o[t] = uint2{w[t][0], w[t][1]};
    if (TERMS < 3) o[t] = bf16_flip(o[t], flip);
  }
}

// planes: term t, real then imaginary part (conj: its negative), ROWS x 32 each
template <bool KC, int TERMS, int ROWS, int NTH>
__device__ inline void chunk_store(unsigned short* P, int tid, const float2 (&v)[ROWS * 4 / NTH][8], bool conj) {
#pragma unroll
  for (int it = 0; it < ROWS * 4 / NTH; ++it) {
    int row, ch;
    chunk_at<KC, ROWS>(tid + it * NTH, row, ch);
    float re[8], im[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      re[j] = v[it][j].x;
      im[j] = v[it][j].y;
    }
    uint4 tr[TERMS], ti[TERMS];
    bf16_terms<TERMS>(re, false, tr);
    bf16_terms<TERMS>(im, conj, ti);
    unsigned short* p = P + plane_at(row, ch);
#pragma unroll
    for (int t = 0; t < TERMS; ++t) {
      *reinterpret_cast<uint4*>(p + (2 * t) * ROWS * BKS) = tr[t];
      *reinterpret_cast<uint4*>(p + (2 * t + 1) * ROWS * BKS) = ti[t];
    }
  }
}

// cr += a_r b_r - a_i b_i, ci += a_r b_i + a_i b_r over a step's 32 k,
// for one row piece and NJ column pieces.  The sign goes to A, or, if the caller
// has more row than column pieces, to b_n = -b_i.
template <int TERMS, int NJ, bool BN = false, class V>
__device__ inline void step_products(const V (&a_r)[TERMS], const V (&a_i)[TERMS], const V (&b_r)[NJ][TERMS],
                                     const V (&b_i)[NJ][TERMS], const V (&b_n)[NJ][TERMS], f4 (&cr)[NJ],
                                     f4 (&ci)[NJ]) {
  // TERMS 3: a step's products are summed on their own and added to the running
  // sums once: a sum over K rounds K / 32 times at its full size instead of
  // 3/8 K times (M x N x K = 20480 x 2048 x 1024: error 1.1e-7 against 7.1e-7
  // with the running sums in the matrix cores and 8.0e-7 on the FP32 matrix
  // cores).  Fewer terms: too few products a step for that.
  constexpr bool APART = TERMS == 3;
  V a_n[TERMS];
#pragma unroll
  for (int t = 0; t < TERMS; ++t) a_n[t] = BN ? a_i[t] : bf16_flip(a_i[t], 0x80008000u);
  f4 xr[NJ], xi[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    xr[j] = APART ? f4{0, 0, 0, 0} : cr[j];
    xi[j] = APART ? f4{0, 0, 0, 0} : ci[j];
  }
#pragma unroll
  for (int g = TERMS - 1; g >= 0; --g)   // the products of 2^-8g, the smallest first
#pragma unroll
    for (int t = 0; t <= g; ++t) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        xr[j] = mfma_bf16(a_r[t], b_r[j][g - t], xr[j]);
        xi[j] = mfma_bf16(a_r[t], b_i[j][g - t], xi[j]);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        xr[j] = mfma_bf16(a_n[t], BN ? b_n[j][g - t] : b_i[j][g - t], xr[j]);
        xi[j] = mfma_bf16(a_i[t], b_r[j][g - t], xi[j]);
      }
    }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    cr[j] = APART ? cr[j] + xr[j] : xr[j];
    ci[j] = APART ? ci[j] + xi[j] : xi[j];
  }
}

// Tile TM x TN, WM x WN waves.  MAPPED: block-sparse work items (or the dense
// grid) with sub-blocks of the tile; otherwise the dense grid only, without
// the branches on a piece's place.
template <int TERMS_, int TM_, int TN_, int WM_, int WN_, int OCC_, bool MAPPED_ = false, bool WIDE_ = false>
struct SplitTile {
  static constexpr int TERMS = TERMS_, TM = TM_, TN = TN_, WM = WM_, WN = WN_, OCC = OCC_, NTH = WM * WN * 64;
  static constexpr bool MAPPED = MAPPED_, WIDE = WIDE_;
};

// Three terms: an infinity, or a number or sum that the scale takes to one, has
// none (h - x is not finite).  Such elements of a wave (a bit each in `again`, (i
// SJ + j) 4 + r) are formed again from the operands themselves, a row of 16 x 16
// pieces at a time on the FP32 matrix cores (v_mfma_f32_16x16x4f32, outputs as
// the BF16 one), in the 3M form of the FP64 kernel, U steps of four k in flight.
// 2048 x 2048 x 1024: all elements again 550 us, a column of B 230 to 460,
// none 174 (a lane per element: 8470; the FP32 matrix cores alone: 278).
struct Again {
  const float2 *A, *B;
  float2* C;
  long long lda, ldb, ldc;
  KIter kr;
  int m0, n0;           // the tile's first row and column in C
  int r0, r1, c0, c1;   // the tile's rows and columns that are there
  int ro, co;           // the wave's first in the tile
  int conj;
  float ar, ai, br, bi;
};
template <bool TA, bool TB, int SI, int SJ>
__device__ inline void form_again(const Again w, unsigned again) {
  constexpr int U = 4;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const float ca = (w.conj & 1) ? -1.f : 1.f, cb = (w.conj & 2) ? -1.f : 1.f;
  const bool has_beta = w.br != 0.f || w.bi != 0.f;
#pragma unroll 1
  for (int i = 0; i < SI; ++i) {
    const unsigned mine = again >> (4 * SJ * i) & ((1u << (4 * SJ)) - 1);
    if (!__any(mine != 0)) continue;
    const int rt = w.ro + 16 * i;   // the pieces that a wave has follow one another
    const int am = rt + lr;
    const bool aok = am >= w.r0 && am < w.r1;
    const float2* ap = TA ? w.A + (w.m0 + am) : w.A + (long long)(w.m0 + am) * w.lda;
    f4 p1[SJ], p2[SJ], p3[SJ];
#pragma unroll
    for (int j = 0; j < SJ; ++j) p1[j] = p2[j] = p3[j] = f4{0, 0, 0, 0};
    for (int v = 0; v < w.kr.n; ++v) {
      const int2 I = w.kr.at(v);
      for (int k = I.x; k < I.y; k += 4 * U) {
        float2 a[U], b[U][SJ];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int kk = k + 4 * u + lk;
          const bool in = kk < I.y;
          a[u] = float2{0.f, 0.f};
          if (in && aok) a[u] = TA ? ap[(long long)kk * w.lda] : ap[kk];
#pragma unroll
          for (int j = 0; j < SJ; ++j) {
            const int bn = w.co + 16 * j + lr;
            b[u][j] = float2{0.f, 0.f};
            if (in && bn >= w.c0 && bn < w.c1)
              b[u][j] = TB ? w.B[(long long)(w.n0 + bn) * w.ldb + kk] : w.B[(long long)kk * w.ldb + (w.n0 + bn)];
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float ay = ca * a[u].y, as = a[u].x + ay;
#pragma unroll
          for (int j = 0; j < SJ; ++j) {
            const float by = cb * b[u][j].y;
            p1[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].x, b[u][j].x, p1[j], 0, 0, 0);
            p2[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ay, by, p2[j], 0, 0, 0);
            p3[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(as, b[u][j].x + by, p3[j], 0, 0, 0);
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < SJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int lm = rt + lk * 4 + r, ln = w.co + 16 * j + lr;
        if (mine >> (4 * j + r) & 1) {
          const float xr = p1[j][r] - p2[j][r], xi = p3[j][r] - p1[j][r] - p2[j][r];
          float2* c = w.C + (long long)(w.m0 + lm) * w.ldc + (w.n0 + ln);
          float2 o{w.ar * xr - w.ai * xi, w.ar * xi + w.ai * xr};
          if (has_beta) {
            const float2 old = *c;
            o.x += w.br * old.x - w.bi * old.y;
            o.y += w.br * old.y + w.bi * old.x;
          }
          *c = o;
        }
      }
  }
}

// conj: bit 0 conjugates A, bit 1 conjugates B (on the way into LDS).
template <class TL, bool TA, bool TB, bool BETA, int TAG>
__global__ __launch_bounds__(TL::NTH, TL::OCC) void gemm_split_kernel(
    int M, int N, int K, float ar, float ai, const float* __restrict__ A, long long lda, long long sa,
    const float* __restrict__ B, long long ldb, long long sb, float br, float bi, float* __restrict__ C, long long ldc,
    long long sc, int S, int Kc, long long sps, const int4* __restrict__ kit, const int2* __restrict__ kiv, int conj) {
  constexpr int TERMS = TL::TERMS, TM = TL::TM, TN = TL::TN, WM = TL::WM, WN = TL::WN, NTH = TL::NTH;
  constexpr int SI = TM / WM / 16, SJ = TN / WN / 16, PA = TM * BKS, PB = TN * BKS;
  constexpr bool BN = SI > SJ;
  static_assert(TL::WIDE || ((TM > TN ? TM : TN) * (LD_WIDE - 1) + BKS) * 8 <= (long long)BUF_BYTES,
                "a tile's rows within the buffer");
  __shared__ __attribute__((aligned(16))) unsigned short As[2 * TERMS * PA], Bs[2 * TERMS * PB];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const TileJob job = tile_job<TM, TN>(M, N, K, S, Kc, TL::MAPPED ? kit : nullptr, kiv);
  const int m0 = job.m0, n0 = job.n0, split = job.split;
  const long long bz = job.bz;
  const float2* Ab = reinterpret_cast<const float2*>(A) + bz * sa;
  const float2* Bb = reinterpret_cast<const float2*>(B) + bz * sb;
  float2* Cb = reinterpret_cast<float2*>(C) + bz * sc + split * sps;

  float2 va[TM * 4 / NTH][8], vb[TN * 4 / NTH][8];
  unsigned oa[TM * 4 / NTH], ob[TN * 4 / NTH];
  chunk_offsets<!TA, TM, NTH>(lda, m0, M, tid, oa, job.r0, job.r1);
  chunk_offsets<TB, TN, NTH>(ldb, n0, N, tid, ob, job.c0, job.c1);
  auto load = [&](int k0, int kend) {
    chunk_load<!TA, TL::WIDE, TM, NTH>(Ab, lda, m0, M, k0, kend, tid, oa, va, job.r0, job.r1);
    chunk_load<TB, TL::WIDE, TN, NTH>(Bb, ldb, n0, N, k0, kend, tid, ob, vb, job.c0, job.c1);
  };

  f4 cr[SI][SJ], ci[SI][SJ];
#pragma unroll
  for (int i = 0; i < SI; ++i)
#pragma unroll
    for (int j = 0; j < SJ; ++j) {
      cr[i][j] = f4{0, 0, 0, 0};
      ci[i][j] = f4{0, 0, 0, 0};
    }

  const int lr = lane & 15, lk = lane >> 4;
  int ro[SI], co[SJ], ni = SI, nj = SJ;
#pragma unroll
  for (int i = 0; i < SI; ++i) ro[i] = wm * (TM / WM) + i * 16;
#pragma unroll
  for (int j = 0; j < SJ; ++j) co[j] = wn * (TN / WN) + j * 16;
  if constexpr (TL::MAPPED) deal_pieces(job, kit != nullptr, wave, ro, co, ni, nj);

  const KIter kr_ = job.kr;
  int iv = 0, k0 = 0, kend = 0;
  if (kr_.n > 0) {
    const int2 I0 = kr_.at(0);
    k0 = I0.x;
    kend = I0.y;
    load(k0, kend);
  }
  const int la = plane_at(lr, lk);   // rows ro + lr, ro a multiple of 16
  for (bool go = kr_.n > 0; go;) {
    int nk0 = k0 + BKS, nkend = kend, niv = iv;
    if (nk0 >= kend) {
      ++niv;
      if (niv < kr_.n) {
        const int2 J = kr_.at(niv);
        nk0 = J.x;
        nkend = J.y;
      }
    }
    const bool more = niv < kr_.n;
    chunk_store<!TA, TERMS, TM, NTH>(As, tid, va, conj & 1);
    chunk_store<TB, TERMS, TN, NTH>(Bs, tid, vb, conj & 2);
    __syncthreads();
    if (more) load(nk0, nkend);   // in flight while this step is multiplied
    uint4 b_r[SJ][TERMS], b_i[SJ][TERMS], b_n[SJ][TERMS];
#pragma unroll
    for (int j = 0; j < SJ; ++j)
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
        b_r[j][t] = *reinterpret_cast<const uint4*>(Bs + (2 * t) * PB + co[j] * BKS + la);
        b_i[j][t] = *reinterpret_cast<const uint4*>(Bs + (2 * t + 1) * PB + co[j] * BKS + la);
        b_n[j][t] = BN ? bf16_flip(b_i[j][t], 0x80008000u) : b_i[j][t];
      }
    // the CU's other workgroup converts its next step meanwhile
    if constexpr (TERMS == 3) __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      if (TL::MAPPED && i >= ni) break;
      uint4 a_r[TERMS], a_i[TERMS];
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
        a_r[t] = *reinterpret_cast<const uint4*>(As + (2 * t) * PA + ro[i] * BKS + la);
        a_i[t] = *reinterpret_cast<const uint4*>(As + (2 * t + 1) * PA + ro[i] * BKS + la);
      }
      if (!TL::MAPPED || nj == SJ)
        step_products<TERMS, SJ, BN>(a_r, a_i, b_r, b_i, b_n, cr[i], ci[i]);
      else if (nj == 1)
        step_products<TERMS, 1, BN>(a_r, a_i, reinterpret_cast<uint4(&)[1][TERMS]>(b_r[0]),
                                    reinterpret_cast<uint4(&)[1][TERMS]>(b_i[0]),
                                    reinterpret_cast<uint4(&)[1][TERMS]>(b_n[0]), reinterpret_cast<f4(&)[1]>(cr[i][0]),
                                    reinterpret_cast<f4(&)[1]>(ci[i][0]));
      // one row piece's operands at a time (192 more registers otherwise)
      if constexpr (TERMS == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (TERMS == 3) __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    go = more;
    iv = niv;
    k0 = nk0;
    kend = nkend;
  }

  // No load is in flight any more, which the compiler sees only here: it waits
  // for one between the stores, and so for the stores, otherwise (A k-contiguous,
  // B transposed, 64 x 64 x 40: 8.3 us, so 7.2).
  __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  const float2* c_some = Cb + ((long long)(m0 + job.r0) * ldc + (n0 + job.c0));   // an element that is there
  auto put = [&](float2* c, float xr, float xi, float2 old) {
    float2 o;
    o.x = ar * xr - ai * xi;
    o.y = ar * xi + ai * xr;
    if constexpr (BETA) {
      o.x += br * old.x - bi * old.y;
      o.y += br * old.y + bi * old.x;
    }
    *c = o;
  };
  static_assert(TERMS < 3 || SI * SJ * 4 <= 32, "a bit per element of a lane");
  unsigned again = 0;   // TERMS 3: the elements to be formed again, bit (i SJ + j) 4 + r
#pragma unroll
  for (int i = 0; i < SI; ++i) {
    if (TL::MAPPED && i >= ni) break;
    auto there = [&](int j, int r) {
      const int lm = ro[i] + lk * 4 + r, ln = co[j] + lr;
      return m0 + lm < M && n0 + ln < N && lm >= job.r0 && lm < job.r1 && ln >= job.c0 && ln < job.c1;
    };
    auto c_at = [&](int j, int r) { return Cb + ((long long)(m0 + ro[i] + lk * 4 + r) * ldc + (n0 + co[j] + lr)); };
    // what C held comes in one round trip, not in one an element: no branches
    float2 old[SJ][4];
    if constexpr (BETA) {
#pragma unroll
      for (int j = 0; j < SJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) old[j][r] = *(there(j, r) ? c_at(j, r) : c_some);
    }
#pragma unroll
    for (int j = 0; j < SJ; ++j) {
      if (TL::MAPPED && j >= nj) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (!there(j, r)) continue;
        constexpr float down = TERMS == 3 ? 1.f / (UP3 * UP3) : 1.f;
        const float xr = down * cr[i][j][r], xi = down * ci[i][j][r];
        if (TERMS == 3 && !(__builtin_isfinite(xr) && __builtin_isfinite(xi))) again |= 1u << ((i * SJ + j) * 4 + r);
        else put(c_at(j, r), xr, xi, old[j][r]);
      }
    }
  }
  if constexpr (TERMS == 3)
    form_again<TA, TB, SI, SJ>(Again{Ab, Bb, Cb, lda, ldb, ldc, kr_, m0, n0, job.r0, min(job.r1, M - m0), job.c0,
                                     min(job.c1, N - n0), ro[0], co[0], conj, ar, ai, br, bi},
                               again);
}

// ---------------------------------------------------------------- short products
// Three terms, K of at most 32: one step, so nothing is staged.  Every wave loads
// its SI row pieces in the MFMA layout (lane l: row l % 16, k KL (l / 16) on),
// converts them and multiplies them with NJ column pieces, one after the other:
// the sums of a gemm_split_kernel of one step, the same bits.  What bounds it: the
// store (and, with beta, the load) of C on large outputs, with the vector
// instructions close behind, so C and the operands are addressed by 32-bit offsets
// and a wave looks at its elements one by one only if one is not finite.
// M x N x K (batch), staged / here in us: 8000 x 5000 x 8 97 / 71, with beta 277 /
// 143 (the store alone at 5.5 TB/s: 58); 2000 x 1500 x 16 13.7 / 11.6; 386 x 133 x 8
// (200) 46 / 25; 887 x 2 x 4 (200) 26 / 11; 14 x 304972 x 8 45 / 18.
template <int KL_, int SI_, int NJ_, int WM_, int WN_> struct ShortTile {
  static constexpr int KL = KL_, SI = SI_, NJ = NJ_, WM = WM_, WN = WN_, TM = WM * SI * 16, TN = WN * NJ * 16;
  static_assert(WM * WN == 4 && SI * NJ * 4 <= 32, "four waves; a bit per element of a lane");
  static_assert((TM > TN ? TM : TN) * LD_WIDE * 8 <= (long long)BUF_BYTES, "a tile's rows within the buffer");
};

// A lane's KL numbers of a piece: off is the first one's offset from the
// uniform base x (BUF_BYTES: a row that is not there), left how many of them there are.
template <bool KC, int KL>
__device__ inline void short_load(const float2* __restrict__ x, long long ld, unsigned off, int left, float2 (&v)[KL]) {
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float2*>(x), 0, (int)BUF_BYTES, 0x00020000);
#pragma unroll
  for (int j = 0; j < KL; ++j) {
    const unsigned o = (j < left ? off : BUF_BYTES) + (KC ? 8u * j : 0u);
    v[j] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, KC ? 0 : j * (int)ld * 8, 0));
  }
}
template <int KL, class V>
__device__ inline void short_terms(const float2 (&v)[KL], bool conj, V (&tr)[3], V (&ti)[3]) {
  float re[KL], im[KL];
#pragma unroll
  for (int j = 0; j < KL; ++j) {
    re[j] = v[j].x;
    im[j] = v[j].y;
  }
  bf16_terms<3>(re, false, tr);
  bf16_terms<3>(im, conj, ti);
}

template <class TL, bool TA, bool TB>
__global__ __launch_bounds__(256, 3) void gemm_short_kernel(int M, int N, int K, float ar, float ai,
                                                             const float* __restrict__ A, long long lda, long long sa,
                                                             const float* __restrict__ B, long long ldb, long long sb,
                                                             float br, float bi, float* __restrict__ C, long long ldc,
                                                             long long sc, int conj) {
  constexpr int KL = TL::KL, SI = TL::SI, NJ = TL::NJ;
  using V = std::conditional_t<KL == 8, uint4, uint2>;
  constexpr float down = 1.f / (UP3 * UP3);
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.y * TL::TM + wave / TL::WN * SI * 16, n0 = blockIdx.x * TL::TN + wave % TL::WN * NJ * 16;
  if (m0 >= M || n0 >= N) return;
  const int mr = M - m0, nr = min(N - n0, NJ * 16);   // rows and columns that are there
  const float2* Ab = reinterpret_cast<const float2*>(A) + (long long)blockIdx.z * sa;
  const float2* Bb = reinterpret_cast<const float2*>(B) + (long long)blockIdx.z * sb;
  float2* Cb = reinterpret_cast<float2*>(C) + (long long)blockIdx.z * sc;
  const int left = K - KL * lk;
  // the lane's first entry of a row, from the operand's first row on
  auto at = [&](bool kc, long long ld, int row) {
    return (kc ? (unsigned)row * (unsigned)ld + (unsigned)(KL * lk) : (unsigned)(KL * lk) * (unsigned)ld + row) * 8u;
  };
  const float2 *xa = TA ? Ab + m0 : Ab + (long long)m0 * lda, *xb = TB ? Bb + (long long)n0 * ldb : Bb + n0;
  auto b_off = [&](int j) {
    const int row = j * 16 + lr;
    return row < nr ? at(TB, ldb, row) : BUF_BYTES;
  };
  float2 va[SI][KL], vb[2][KL];
#pragma unroll
  for (int i = 0; i < SI; ++i) {
    const int row = i * 16 + lr;
    short_load<!TA, KL>(xa, lda, row < mr ? at(!TA, lda, row) : BUF_BYTES, left, va[i]);
  }
  short_load<TB, KL>(xb, ldb, b_off(0), left, vb[0]);

  // C from the wave's first element on; row r of a piece is r ldc further
  const __amdgpu_buffer_rsrc_t rc =
      __builtin_amdgcn_make_buffer_rsrc(Cb + ((long long)m0 * ldc + n0), 0, (int)BUF_BYTES, 0x00020000);
  const int lc = (int)ldc * 8;
  const bool has_beta = (br != 0.f) || (bi != 0.f), whole = mr >= SI * 16 && nr >= NJ * 16;
  // the offset of row r = 0 of piece (i, j), past the buffer if element r is not there
  auto c_off = [&](int i, int j, int r) {
    const unsigned o = (unsigned)((i * 16 + lk * 4) * (int)ldc + j * 16 + lr) * 8u;
    return whole || (i * 16 + lk * 4 + r < mr && j * 16 + lr < nr) ? o : BUF_BYTES;
  };
  float2 old[SI][4];
  auto load_c = [&](int j, float2 (&o)[SI][4]) {
#pragma unroll
    for (int i = 0; i < SI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        o[i][r] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rc, (int)c_off(i, j, r), r * lc, 0));
  };

  V a_r[SI][3], a_i[SI][3];
#pragma unroll
  for (int i = 0; i < SI; ++i) short_terms(va[i], conj & 1, a_r[i], a_i[i]);
  unsigned again = 0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j * 16 >= nr) break;
    if (j + 1 < NJ) short_load<TB, KL>(xb, ldb, b_off(j + 1), left, vb[(j + 1) & 1]);
    if (has_beta) load_c(j, old);
    V b_r[1][3], b_i[1][3];
    short_terms(vb[j & 1], conj & 2, b_r[0], b_i[0]);
    f4 cr[SI][1], ci[SI][1];
    float t = 0.f;   // not a zero if one of the sums is not finite
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      cr[i][0] = ci[i][0] = f4{0, 0, 0, 0};
      step_products<3, 1>(a_r[i], a_i[i], b_r, b_i, b_i, cr[i], ci[i]);
#pragma unroll
      for (int r = 0; r < 4; ++r) t = fmaf(cr[i][0][r], 0.f, fmaf(ci[i][0][r], 0.f, t));
    }
    const bool some = __any(!(t == 0.f));
#pragma unroll
    for (int i = 0; i < SI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float xr = down * cr[i][0][r], xi = down * ci[i][0][r];
        f2v o;
        o.x = ar * xr - ai * xi;
        o.y = ar * xi + ai * xr;
        if (has_beta) {
          const float2 c = old[i][r];
          o.x += br * c.x - bi * c.y;
          o.y += br * c.y + bi * c.x;
        }
        unsigned off = c_off(i, j, r);
        if (some && !(__builtin_isfinite(xr) && __builtin_isfinite(xi))) {
          if (off != BUF_BYTES) again |= 1u << ((i * NJ + j) * 4 + r);
          off = BUF_BYTES;
        }
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, o), rc, (int)off, r * lc, 0);
      }
  }
  KIter all;
  all.iv = nullptr;
  all.n = 1;
  all.one = make_int2(0, K);
  form_again<TA, TB, SI, NJ>(
      Again{Ab, Bb, Cb, lda, ldb, ldc, all, m0, n0, 0, min(SI * 16, mr), 0, nr, 0, 0, conj, ar, ai, br, bi}, again);
}

// ---------------------------------------------------------------- term images
// For one and two terms the conversion costs more than the products: a large
// operand entry is converted once per output tile of its row or column.  With
// scratch at hand the terms are written once, as the LDS blocks that the
// product stages, and loaded straight into LDS (no registers, no address
// arithmetic).  Three terms: the product takes as long either way (six products
// an entry, 1.2 PFLOP/s), so it keeps the conversion on the way in.
// 14000 x 2048 x 1021, TERMS 1: 497 us -> 43 of conversion and 196, 1.2
// PFLOP/s; 10752 x 1402 x 768, TERMS 2: 310 -> 27 and 218, 1.28 PFLOP/s in BF16
// (a large library product in plain BF16 reaches 1.21 here).
//
// Block (64 rows, 32 k): the 2 TERMS planes (term t, real, imaginary) one
// after the other, each as plane_at; the k blocks of 64 rows follow one
// another.  Rows and k past the operand are zeros.
constexpr int IROWS = 64;
template <int TERMS> constexpr int IBLOCK = 2 * TERMS * IROWS * BKS;   // numbers of a block

// grid (k blocks, row blocks), a chunk a thread: a wave loads whole 128-byte
// lines in either order and stores a plane's 16 rows, 1 KiB
template <bool KC, int TERMS>
__global__ __launch_bounds__(256) void terms_kernel(const float* __restrict__ X, long long ld, int R, int K, int conj,
                                                    unsigned short* __restrict__ img) {
  const int lane = threadIdx.x & 63, row = (threadIdx.x >> 6) * 16 + (KC ? lane >> 2 : lane & 15);
  const int ch = KC ? lane & 3 : lane >> 4;
  const long long r = (long long)blockIdx.y * IROWS + row;
  const int k = blockIdx.x * BKS + 8 * ch;
  float re[8], im[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) re[j] = im[j] = 0.f;
  if (r < R && k < K) {
    const float2* x = reinterpret_cast<const float2*>(X) + (KC ? r * ld + k : (long long)k * ld + r);
    if (KC && k + 8 <= K) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f4u t = reinterpret_cast<const f4u*>(x)[j];
        re[2 * j] = t.x;
        im[2 * j] = t.y;
        re[2 * j + 1] = t.z;
        im[2 * j + 1] = t.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (k + j < K) {
          const float2 t = KC ? x[j] : x[j * ld];
          re[j] = t.x;
          im[j] = t.y;
        }
    }
  }
  uint4 tr[TERMS], ti[TERMS];
  bf16_terms<TERMS>(re, false, tr);
  bf16_terms<TERMS>(im, conj, ti);
  unsigned short* o = img + ((long long)blockIdx.y * gridDim.x + blockIdx.x) * IBLOCK<TERMS> + plane_at(row, ch);
#pragma unroll
  for (int t = 0; t < TERMS; ++t) {
    *reinterpret_cast<uint4*>(o + (2 * t) * IROWS * BKS) = tr[t];
    *reinterpret_cast<uint4*>(o + (2 * t + 1) * IROWS * BKS) = ti[t];
  }
}

// blocks r0 / 64 .. of an image's k block into LDS, 1 KiB a wave and load
template <int TERMS, int ROWS, int NTH>
__device__ inline void image_load(const unsigned short* __restrict__ img, int nkc, int r0, int k0, unsigned short* P,
                                  int wave, int lane) {
  constexpr int PER = IBLOCK<TERMS> / 512, PIECES = ROWS / IROWS * PER, NW = NTH / 64;
  static_assert(ROWS % IROWS == 0 && PIECES % NW == 0);
#pragma unroll
  for (int it = 0; it < PIECES / NW; ++it) {
    const int piece = wave + it * NW;
    const unsigned short* g = img + ((long long)(r0 / IROWS + piece / PER) * nkc + k0 / BKS) * IBLOCK<TERMS> +
                              piece % PER * 512 + lane * 8;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)(P + piece * 512), 16, 0, 0);
  }
}

// Tile TM x TN, WM x WN waves, OCC workgroups of them a CU at four waves each.
// STAGES 2: the next step's blocks arrive in a second buffer; 1: the step's
// last reads are waited for first, and the CU's other workgroups multiply
// meanwhile.  Tiles are dealt GROUP rows at a time, down the rows first: the
// workgroups that run together on an XCD share both panels (14000 x 2048 x
// 1021, TERMS 1: 196 us; along the rows 215).
template <int TERMS_, int TM_, int TN_, int WM_, int WN_, int STAGES_, int OCC_>
struct ImageTile {
  static constexpr int TERMS = TERMS_, TM = TM_, TN = TN_, WM = WM_, WN = WN_, STAGES = STAGES_, OCC = OCC_;
  static constexpr int NTH = WM * WN * 64, GROUP = 8;
};

// IA, IB: images of op(A) (rows m) and op(B) (rows n) of nkc k blocks, padded to
// whole tiles by the host.  Split s of S takes k from s Kc.
template <class TL, bool BETA>
__global__ __launch_bounds__(TL::NTH, TL::OCC) void gemm_image_kernel(
    int M, int N, int K, float ar, float ai, const unsigned short* __restrict__ IA,
    const unsigned short* __restrict__ IB, int nkc, float br, float bi, float* __restrict__ C, long long ldc, int S,
    int Kc, long long sps) {
  constexpr int TERMS = TL::TERMS, TM = TL::TM, TN = TL::TN, WM = TL::WM, WN = TL::WN, NTH = TL::NTH;
  constexpr int SI = TM / WM / 16, SJ = TN / WN / 16, PA = 2 * TERMS * TM * BKS, PB = 2 * TERMS * TN * BKS;
  // buffers of their own: a read of one does not wait for the loads into the other
  __shared__ __attribute__((aligned(16))) unsigned short P0[PA + PB], P1[TL::STAGES == 2 ? PA + PB : 8];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const TileJob job = tile_job<TM, TN>(M, N, K, S, Kc, nullptr, nullptr);
  const int gx = gridDim.x, gy = gridDim.y, lin = (job.m0 / TM) * gx + job.n0 / TN;
  const int g0 = lin / (TL::GROUP * gx) * TL::GROUP, rows = min(TL::GROUP, gy - g0), in = lin - g0 * gx;
  const int m0 = (g0 + in % rows) * TM, n0 = in / rows * TN;
  const int kb = job.kr.one.x, ke = job.kr.one.y;
  float2* Cb = reinterpret_cast<float2*>(C) + job.split * sps;

  f4 cr[SI][SJ], ci[SI][SJ];
#pragma unroll
  for (int i = 0; i < SI; ++i)
#pragma unroll
    for (int j = 0; j < SJ; ++j) cr[i][j] = ci[i][j] = f4{0, 0, 0, 0};

  const int lr = lane & 15, lk = lane >> 4, la = plane_at(lr, lk);
  auto load = [&](int k, unsigned short* P) {
    image_load<TERMS, TM, NTH>(IA, nkc, m0, k, P, wave, lane);
    image_load<TERMS, TN, NTH>(IB, nkc, n0, k, P + PA, wave, lane);
  };
  auto at = [&](const unsigned short* P, int t, int r) {
    return *reinterpret_cast<const uint4*>(P + (r / IROWS) * IBLOCK<TERMS> + (t * IROWS + r % IROWS) * BKS + la);
  };
  auto landed = [] {
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's blocks are in LDS
    __syncthreads();
  };
  auto step = [&](const unsigned short* P, unsigned short* next, int k) {
    if (TL::STAGES == 2 && k + BKS < ke) load(k + BKS, next);
    uint4 b_r[SJ][TERMS], b_i[SJ][TERMS];
#pragma unroll
    for (int j = 0; j < SJ; ++j)
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
        b_r[j][t] = at(P + PA, 2 * t, wn * (TN / WN) + j * 16);
        b_i[j][t] = at(P + PA, 2 * t + 1, wn * (TN / WN) + j * 16);
      }
#pragma unroll
    for (int i = 0; i < SI; ++i) {
      uint4 a_r[TERMS], a_i[TERMS];
#pragma unroll
      for (int t = 0; t < TERMS; ++t) {
        a_r[t] = at(P, 2 * t, wm * (TM / WM) + i * 16);
        a_i[t] = at(P, 2 * t + 1, wm * (TM / WM) + i * 16);
      }
      if (TL::STAGES == 1 && i + 1 == SI) {
        __syncthreads();   // every wave has read its blocks
        if (k + BKS < ke) load(k + BKS, next);
        __builtin_amdgcn_sched_barrier(0);
      }
      step_products<TERMS, SJ>(a_r, a_i, b_r, b_i, b_i, cr[i], ci[i]);
    }
    landed();
  };
  if (kb < ke) {
    load(kb, P0);
    landed();
    if constexpr (TL::STAGES == 1) {
      for (int k = kb; k < ke; k += BKS) step(P0, P0, k);
    } else {
      for (int k = kb; k < ke; k += 2 * BKS) {
        step(P0, P1, k);
        if (k + BKS < ke) step(P1, P0, k + BKS);
      }
    }
  }

#pragma unroll
  for (int i = 0; i < SI; ++i) {
    const int gm0 = m0 + wm * (TM / WM) + i * 16 + lk * 4, gn0 = n0 + wn * (TN / WN) + lr;
    auto there = [&](int j, int r) { return gm0 + r < M && gn0 + j * 16 < N; };
    auto c_at = [&](int j, int r) { return Cb + ((long long)(gm0 + r) * ldc + (gn0 + j * 16)); };
    float2 old[SJ][4];   // what C held, in one round trip
    if constexpr (BETA) {
#pragma unroll
      for (int j = 0; j < SJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) old[j][r] = *(there(j, r) ? c_at(j, r) : Cb + ((long long)m0 * ldc + n0));
    }
#pragma unroll
    for (int j = 0; j < SJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (!there(j, r)) continue;
        const float xr = cr[i][j][r], xi = ci[i][j][r];
        float2 o;
        o.x = ar * xr - ai * xi;
        o.y = ar * xi + ai * xr;
        if constexpr (BETA) {
          o.x += br * old[j][r].x - bi * old[j][r].y;
          o.y += br * old[j][r].y + bi * old[j][r].x;
        }
        *c_at(j, r) = o;
      }
  }
}

// ---------------------------------------------------------------- FP64 GEMM
// An FP64 MFMA takes 64 cycles for 1 KiB of operands, so the vector caches can
// feed the matrix cores by themselves: every wave loads its operand pieces
// straight in the MFMA layout (lane l: row or column l % 16, k = l / 16) PF
// steps of four k ahead, nothing passes through LDS and no wave waits for
// another.  A block is WM x WN waves of SI x SJ 16 x 16 pieces each, times up
// to PARTS waves that take one part of K each and meet in LDS at the end.
// A complex product is three real ones (the 3M form): p1 = sum ar br,
// p2 = sum ai bi, p3 = sum (ar + ai)(br + bi); Re = p1 - p2, Im = p3 - p1 - p2.
// The parts of K depend on M, N and K alone (choose_splits) and are summed in
// their order, so every tile gives the same bits.
// What bounds it: the matrix cores (80 ns a piece and step) and, not quite
// beside them, the operand loads (5 us a MiB and CU with two or more waves on
// a SIMD, 9 with one).  20480 x 2048 x 1024: 4.02 ms, 85 TFLOP/s at 8 a
// complex multiply-add, 82% of what three products allow (through LDS tiles
// with a barrier a step: 4.47 ms).
template <int SI_, int SJ_, int WM_, int WN_, int PARTS_, int PF_, bool MAPPED_ = false, bool WIDE_ = false>
struct DirectTile {
  static constexpr int SI = SI_, SJ = SJ_, WM = WM_, WN = WN_, PARTS = PARTS_, PF = PF_;
  static constexpr int TM = WM * SI * 16, TN = WN * SJ * 16, NTH = WM * WN * PARTS * 64;
  static constexpr bool MAPPED = MAPPED_, WIDE = WIDE_;
  static_assert(PARTS == 1 || WM * WN == 1, "waves along K or over the tile");
};
constexpr long long LD_WIDE64 = 1LL << 21;   // 64 rows of 2^21 complex128: 2^31 bytes

// An operand as a wave reads it: rows (columns of B) r0 + off, lane row
// off + l % 16.  KC: k is the contiguous index.
template <bool KC, bool WIDE, int NP> struct DirectOperand {
  const double2* base;   // row r0, k = 0
  long long ld;
  unsigned at[NP];       // byte offset of the lane's entry at the step's first k
  int row[NP];           // WIDE: the lane's row, -1 if it is not there
  __device__ void init(const double2* X, long long ld_, int r0, int R, const int (&off)[NP], int lo, int hi, int lr,
                       int lk) {
    ld = ld_;
    base = X + (KC ? (long long)r0 * ld : (long long)r0);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int r = off[i] + lr;
      const bool in = r0 + r < R && r >= lo && r < hi;
      if constexpr (WIDE) row[i] = in ? r : -1;
      else at[i] = in ? (KC ? (unsigned)r * (unsigned)ld + lk : (unsigned)lk * (unsigned)ld + r) * 16u : BUF_BYTES;
    }
  }
  // the first N pieces
  template <int N> __device__ void load(int k0, bool in, int lk, double2 (&v)[NP]) const {
    if constexpr (WIDE) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        v[i] = double2{0.0, 0.0};
        if (in && row[i] >= 0)
          v[i] = base[KC ? (long long)row[i] * ld + k0 + lk : (long long)(k0 + lk) * ld + row[i]];
      }
    } else {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<double2*>(base + (KC ? (long long)k0 : (long long)k0 * ld)), 0, (int)BUF_BYTES, 0x00020000);
#pragma unroll
      for (int i = 0; i < N; ++i)
        v[i] = __builtin_bit_cast(double2,
                                  __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(in ? at[i] : BUF_BYTES), 0, 0));
    }
  }
};

// S splits over the grid, or (PARTS > 1) a block's waves as parts of Kc each;
// conj: bit 0 conjugates A, bit 1 conjugates B
template <class TL, bool TA, bool TB, bool BETA, int TAG>
__global__ __launch_bounds__(TL::NTH, TL::NTH > 512 ? 4 : 2) void gemm_direct_kernel(
    int M, int N, int K, double ar, double ai, const double* __restrict__ A, long long lda, long long sa,
    const double* __restrict__ B, long long ldb, long long sb, double br, double bi, double* __restrict__ C,
    long long ldc, long long sc, int S, int Kc, long long sps, const int4* __restrict__ kit,
    const int2* __restrict__ kiv, int conj) {
  constexpr int SI = TL::SI, SJ = TL::SJ, WN = TL::WN, PF = TL::PF, E = SI * SJ * 4;
  static_assert(TL::WIDE || ((TL::TM > TL::TN ? TL::TM : TL::TN) * (LD_WIDE64 - 1) + 4) * 16 <= (long long)BUF_BYTES,
                "a tile's rows within the buffer");
  extern __shared__ unsigned char direct_lds[];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int parts = TL::PARTS > 1 ? (int)(blockDim.x >> 6) : 1;
  const int wk = TL::PARTS > 1 ? wave : 0, wmn = TL::PARTS > 1 ? 0 : wave;
  const TileJob job = tile_job<TL::TM, TL::TN>(M, N, K, S, TL::PARTS > 1 ? K : Kc, TL::MAPPED ? kit : nullptr, kiv);
  // the wave's pieces: the product of ni rows and nj columns of pieces at the
  // tile offsets ro, co
  int ro[SI], co[SJ], ni = SI, nj = SJ;
#pragma unroll
  for (int i = 0; i < SI; ++i) ro[i] = (wmn / WN * SI + i) * 16;
#pragma unroll
  for (int j = 0; j < SJ; ++j) co[j] = (wmn % WN * SJ + j) * 16;
  if constexpr (TL::MAPPED) {
    deal_pieces(job, kit != nullptr, wmn, ro, co, ni, nj);
    if (ni == 0 || nj == 0) return;
  }

  DirectOperand<!TA, TL::WIDE, SI> oa;
  DirectOperand<TB, TL::WIDE, SJ> ob;
  oa.init(reinterpret_cast<const double2*>(A) + job.bz * sa, lda, job.m0, M, ro, job.r0, job.r1, lr, lk);
  ob.init(reinterpret_cast<const double2*>(B) + job.bz * sb, ldb, job.n0, N, co, job.c0, job.c1, lr, lk);

  d4 p1[SI][SJ], p2[SI][SJ], p3[SI][SJ];
#pragma unroll
  for (int i = 0; i < SI; ++i)
#pragma unroll
    for (int j = 0; j < SJ; ++j) p1[i][j] = p2[i][j] = p3[i][j] = d4{0, 0, 0, 0};
  const double ca = (conj & 1) ? -1.0 : 1.0, cb = (conj & 2) ? -1.0 : 1.0;
  const KIter kr = job.kr;
  // the steps over the wave's intervals with NI x NJ pieces, PF of them in
  // flight; `left` counts those loaded and not yet multiplied
  auto multiply = [&](auto ni_, auto nj_) {
    constexpr int NI = decltype(ni_)::value, NJ = decltype(nj_)::value;
    int iv = 0, k = 0, kend = 0, left = 0;
    if (kr.n > 0) {
      const int2 I = kr.at(0);
      k = __builtin_amdgcn_readfirstlane(I.x);
      kend = __builtin_amdgcn_readfirstlane(I.y);
    }
    if (parts > 1) {
      k = wk * Kc;
      kend = min(kend, k + Kc);
    }
    double2 va[PF][SI], vb[PF][SJ];
    auto load = [&](double2 (&a)[SI], double2 (&b)[SJ]) {
      if constexpr (TL::MAPPED) {
        while (k >= kend && ++iv < kr.n) {
          const int2 I = kr.at(iv);
          k = __builtin_amdgcn_readfirstlane(I.x);
          kend = __builtin_amdgcn_readfirstlane(I.y);
        }
      }
      if (k >= kend) return;
      const bool in = k + lk < kend;
      oa.template load<NI>(k, in, lk, a);
      ob.template load<NJ>(k, in, lk, b);
      k += 4;
      ++left;
    };
#pragma unroll
    for (int p = 0; p < PF; ++p) load(va[p], vb[p]);
    while (left > 0) {
#pragma unroll
      for (int p = 0; p < PF; ++p) {
        if (left <= 0) break;
        double as[NI], bs[NJ];
#pragma unroll
        for (int i = 0; i < NI; ++i) as[i] = fma(ca, va[p][i].y, va[p][i].x);
#pragma unroll
        for (int j = 0; j < NJ; ++j) bs[j] = fma(cb, vb[p][j].y, vb[p][j].x);
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            p1[i][j] = mfma(va[p][i].x, vb[p][j].x, p1[i][j]);
            p2[i][j] = mfma(va[p][i].y, vb[p][j].y, p2[i][j]);
            p3[i][j] = mfma(as[i], bs[j], p3[i][j]);
          }
        --left;
        load(va[p], vb[p]);
      }
    }
  };
  if constexpr (TL::MAPPED) {
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    if (ni == 2 && nj == 2) multiply(Two{}, Two{});
    else if (ni == 2) multiply(Two{}, One{});
    else if (nj == 2) multiply(One{}, Two{});
    else multiply(One{}, One{});
  } else {
    multiply(std::integral_constant<int, SI>{}, std::integral_constant<int, SJ>{});
  }
  // p2 holds the product of the stored imaginary parts
  double2 x[E];
#pragma unroll
  for (int i = 0; i < SI; ++i)
#pragma unroll
    for (int j = 0; j < SJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double q1 = p1[i][j][r], q2 = ca * cb * p2[i][j][r];
        x[(i * SJ + j) * 4 + r] = double2{q1 - q2, p3[i][j][r] - q1 - q2};
      }
  double2* red = reinterpret_cast<double2*>(direct_lds) + lane;   // [part][entry][lane]
  if (parts > 1) {
#pragma unroll
    for (int e = 0; e < E; ++e) red[(wk * E + e) * 64] = x[e];
    __syncthreads();
  }
  double2* Cb = reinterpret_cast<double2*>(C) + job.bz * sc + job.split * sps;
  // row of the MFMA's result r: lane / 16 + 4 r, column lane % 16
  auto there = [&](int e) {
    const int lm = ro[e / 4 / SJ] + lk + 4 * (e % 4), ln = co[e / 4 % SJ] + lr;
    return job.m0 + lm < M && job.n0 + ln < N && lm >= job.r0 && lm < job.r1 && ln >= job.c0 && ln < job.c1;
  };
  auto c_at = [&](int e) {
    return Cb + ((long long)(job.m0 + ro[e / 4 / SJ] + lk + 4 * (e % 4)) * ldc + (job.n0 + co[e / 4 % SJ] + lr));
  };
  const double2* c_some = Cb + ((long long)(job.m0 + job.r0) * ldc + (job.n0 + job.c0));   // an element that is there
  // the entry's sum over the parts
  auto sum = [&](int e) {
    double2 v = x[e];
    if (parts > 1) {
      v = double2{0.0, 0.0};
      for (int w = 0; w < parts; ++w) {
        const double2 u = red[(w * E + e) * 64];
        v.x += u.x;
        v.y += u.y;
      }
    }
    return v;
  };
  auto mine = [&](int e) {   // the parts' waves share the sums and stores
    return e / 4 / SJ < ni && e / 4 % SJ < nj && (parts == 1 || e % parts == wk);
  };
  if constexpr (!BETA) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if (!mine(e)) continue;
      const double2 v = sum(e);
      if (there(e)) *c_at(e) = double2{ar * v.x - ai * v.y, ar * v.y + ai * v.x};
    }
    return;
  }
  constexpr int G = E < 8 ? E : 8;
#pragma unroll
  for (int e0 = 0; e0 < E; e0 += G) {
    // what C held comes in one round trip, not in one an entry: no branches
    double2 old[G];
#pragma unroll
    for (int g = 0; g < G; ++g) old[g] = *(there(e0 + g) ? c_at(e0 + g) : c_some);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int e = e0 + g;
      if (!mine(e)) continue;
      const double2 v = sum(e);
      double2 o{ar * v.x - ai * v.y, ar * v.y + ai * v.x};
      o.x += br * old[g].x - bi * old[g].y;
      o.y += br * old[g].y + bi * old[g].x;
      if (there(e)) *c_at(e) = o;
    }
  }
}

// Deterministic split-K reduction: C = alpha * sum_s P[s] + beta * C.
template <typename T>
__global__ void splitk_reduce_kernel(const T* __restrict__ P, int S, long long M, long long N, T ar, T ai,
                                     T br, T bi, T* __restrict__ C, long long ldc) {
  using c2 = typename VT<T>::c2;
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= M * N) return;
  const c2* Pc = reinterpret_cast<const c2*>(P);
  T xr = T(0), xi = T(0);
  for (int s = 0; s < S; ++s) {
    const c2 v = Pc[(long long)s * M * N + idx];
    xr += v.x;
    xi += v.y;
  }
  const long long m = idx / N, n = idx % N;
  c2* Cc = reinterpret_cast<c2*>(C);
  c2 o;
  o.x = ar * xr - ai * xi;
  o.y = ar * xi + ai * xr;
  if (br != T(0) || bi != T(0)) {
    const c2 old = Cc[m * ldc + n];
    o.x += br * old.x - bi * old.y;
    o.y += br * old.y + bi * old.x;
  }
  Cc[m * ldc + n] = o;
}

// Split-K reduction of a block-sparse product: C[b] = alpha * sum of the
// nonempty parts of each tile + beta * C[b]; the parts are P[s][b][m][n].
template <typename T>
__global__ void splitk_reduce_map_kernel(const T* __restrict__ P, int batch, long long M, long long N, int gx,
                                         const int* __restrict__ tinfo, T ar, T ai, T br, T bi, T* __restrict__ C,
                                         long long ldc, long long sc) {
  using c2 = typename VT<T>::c2;
  const long long MN = M * N;
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= MN * batch) return;
  const long long b = idx / MN, r = idx % MN, m = r / N, n = r % N;
  const long long tiles = ((M + BM - 1) / BM) * (long long)gx;
  const int* ti = tinfo + 6 * (b * tiles + (m / BM) * gx + n / BN);
  const int ns = ti[2 + ((m % BM) >= ti[0] ? 2 : 0) + ((n % BN) >= ti[1] ? 1 : 0)];
  const c2* Pc = reinterpret_cast<const c2*>(P);
  T xr = T(0), xi = T(0);
  for (int s = 0; s < ns; ++s) {
    const c2 v = Pc[(long long)s * batch * MN + idx];
    xr += v.x;
    xi += v.y;
  }
  c2* Cc = reinterpret_cast<c2*>(C) + b * sc + m * ldc + n;
  c2 o;
  o.x = ar * xr - ai * xi;
  o.y = ar * xi + ai * xr;
  if (br != T(0) || bi != T(0)) {
    const c2 old = *Cc;
    o.x += br * old.x - bi * old.y;
    o.y += br * old.y + bi * old.x;
  }
  *Cc = o;
}

// Compute mode of the complex64 GEMMs on the calling host thread (kern::set_float_mode):
// 0 FP32 (three BF16 terms), 1 BF16, 2 two BF16 terms.
thread_local int tl_float_mode = 0;

// block-sparse map of the next product issued from the calling host thread
thread_local const kern::KMap* tl_kmap = nullptr;

// One product as its kernels take it.
template <typename T> struct Product {
  hipStream_t s;
  int M, N, K, batch;
  const T* A;
  long long lda, sa;
  const T* B;
  long long ldb, sb;
  T* C;
  long long ldc, sc;
  T ar, ai, br, bi;
  void* ws;
  size_t ws_bytes;
};

// Tiles of the BF16-term products, the largest first, with the time of one
// 32-wide K step of a workgroup in us: alone on its CU, and its share when
// the CU's other workgroups keep it busy (20480 x 2048 x 1024, 4096 x 509 x
// 512).  A larger tile converts and reads each operand entry fewer times and
// so costs less per output, a smaller one fills the 256 CUs on smaller
// outputs: complete products of 20480 x 2048 x 1024 / 4096 x 509 x 512 take,
// largest to smallest tile, TERMS 3: 1850 / 68, 2020 / 52 us; TERMS 2: 1165 /
// 50, 1370 / 41 us; TERMS 1: 583 / 45, 663 / 29, 895 / 27 us.
struct TileCost {
  int tm, tn;
  double alone, shared;
};
template <int TERMS> struct SplitTiles;
template <> struct SplitTiles<3> {
  static constexpr int n = 2;
  static constexpr TileCost cost[n] = {{128, 64, 3.9, 2.9}, {64, 64, 2.2, 1.55}};
  using T0 = SplitTile<3, 128, 64, 2, 2, 2>;
  using T1 = T0;
  using Small = SplitTile<3, 64, 64, 2, 2, 2>;
  using Mapped = SplitTile<3, 64, 64, 2, 2, 2, true>;
  using Wide = SplitTile<3, 64, 64, 2, 2, 2, true, true>;
};
template <> struct SplitTiles<2> {
  static constexpr int n = 2;
  static constexpr TileCost cost[n] = {{128, 128, 2.9, 3.65}, {64, 64, 1.6, 1.05}};
  using T0 = SplitTile<2, 128, 128, 2, 4, 2>;
  using T1 = T0;
  using Small = SplitTile<2, 64, 64, 2, 2, 3>;
  using Mapped = SplitTile<2, 64, 64, 2, 2, 3, true>;
  using Wide = SplitTile<2, 64, 64, 2, 2, 2, true, true>;
};
template <> struct SplitTiles<1> {
  static constexpr int n = 3;
  static constexpr TileCost cost[n] = {{256, 128, 2.7, 3.5}, {128, 128, 1.8, 2.05}, {64, 64, 1.1, 0.69}};
  using T0 = SplitTile<1, 256, 128, 4, 2, 1>;
  using T1 = SplitTile<1, 128, 128, 4, 2, 2>;
  using Small = SplitTile<1, 64, 64, 2, 2, 3>;
  using Mapped = SplitTile<1, 64, 64, 2, 2, 3, true>;
  using Wide = SplitTile<1, 64, 64, 2, 2, 2, true, true>;
};

template <class TL, bool TA, bool TB, int TAG>
void launch_split_tile(dim3 grid, const Product<float>& p, float* C, long long ldc, long long sc, bool plain, int S,
                       int Kc, long long sps, const int4* kit, const int2* kiv, int conj) {
  auto go = [&](auto beta) {
    hipLaunchKernelGGL((gemm_split_kernel<TL, TA, TB, decltype(beta)::value, TAG>), grid, dim3(TL::NTH), 0, p.s, p.M,
                       p.N, p.K, plain ? 1.f : p.ar, plain ? 0.f : p.ai, p.A, p.lda, p.sa, p.B, p.ldb, p.sb,
                       plain ? 0.f : p.br, plain ? 0.f : p.bi, C, ldc, sc, S, Kc, sps, kit, kiv, conj);
  };
  if (plain || (p.br == 0.f && p.bi == 0.f)) go(std::false_type{});
  else go(std::true_type{});
}

// Which products are short.  Staged / short in us: 3752 x 3222 x 24 32.5 / 32, 8000 x
// 5000 x 24 106 / 98, x 32 102 / 108, 2000 x 1500 x 32 13.3 / 15; but 700 x 700 x 32
// 7.3 / 6.3, 14 x 304972 x 32 43 / 27.  Up to K = 16 a lane holds four k (v_mfma 16 x
// 16 x 16: half the numbers to convert), from 17 on eight.
inline bool short_product(const Product<float>& p) {
  if (p.K < 1 || wide_ld(p.lda, p.ldb, LD_WIDE) || wide_ld(p.ldc, p.ldc, LD_WIDE)) return false;
  return p.K <= 24 || (p.K <= 32 && (p.M <= 16 || p.N <= 16 || (double)p.M * p.N * p.batch < 1e6));
}

template <bool TA, bool TB> void launch_short(const Product<float>& p, int conj) {
  auto go = [&](auto tl) {
    using TL = decltype(tl);
    const dim3 grid((p.N + TL::TN - 1) / TL::TN, (p.M + TL::TM - 1) / TL::TM, p.batch);
    hipLaunchKernelGGL((gemm_short_kernel<TL, TA, TB>), grid, dim3(256), 0, p.s, p.M, p.N, p.K, p.ar, p.ai, p.A, p.lda,
                       p.sa, p.B, p.ldb, p.sb, p.br, p.bi, p.C, p.ldc, p.sc, conj);
  };
  auto tile = [&](auto kl) {
    constexpr int KL = decltype(kl)::value;
    const double mn = (double)p.M * p.N * p.batch;
    // narrow and low outputs: tiles as narrow or low
    if (p.N <= 16) go(ShortTile<KL, 2, 1, 4, 1>{});
    else if (p.M <= 16) go(ShortTile<KL, 1, 2, 1, 4>{});
    else if (mn < 1e6) go(ShortTile<KL, 2, 1, 2, 2>{});
    else if (mn < 2e7 || p.N < 1024) go(ShortTile<KL, 2, 2, 2, 2>{});
    else go(ShortTile<KL, 2, 4, 2, 2>{});
  };
  if (p.K <= 16) tile(std::integral_constant<int, 4>{});
  else tile(std::integral_constant<int, 8>{});
}

// kit null: the dense grid on tile `tile` of SplitTiles (S > 1: partial
// products, plain); otherwise a block-sparse map of n_items items.
template <int TERMS, bool TA, bool TB, int TAG>
void launch_split(const Product<float>& p, int conj, int tile, int n_items, float* C, long long ldc, long long sc,
                  bool plain, int S, int Kc, long long sps, const int4* kit, const int2* kiv) {
  using TS = SplitTiles<TERMS>;
  const bool wide = wide_ld(p.lda, p.ldb, LD_WIDE);
  const int tm = wide ? 64 : TS::cost[tile].tm, tn = wide ? 64 : TS::cost[tile].tn;
  const dim3 grid = kit ? dim3(n_items)
                        : dim3((p.N + tn - 1) / tn, (p.M + tm - 1) / tm, S > 1 ? S : p.batch);
  if (wide)
    launch_split_tile<typename TS::Wide, TA, TB, TAG>(grid, p, C, ldc, sc, plain, S, Kc, sps, kit, kiv, conj);
  else if (kit)
    launch_split_tile<typename TS::Mapped, TA, TB, TAG>(grid, p, C, ldc, sc, plain, S, Kc, sps, kit, kiv, conj);
  else if (tile == TS::n - 1)
    launch_split_tile<typename TS::Small, TA, TB, TAG>(grid, p, C, ldc, sc, plain, S, Kc, sps, kit, kiv, conj);
  else if (tile == 0)
    launch_split_tile<typename TS::T0, TA, TB, TAG>(grid, p, C, ldc, sc, plain, S, Kc, sps, kit, kiv, conj);
  else
    launch_split_tile<typename TS::T1, TA, TB, TAG>(grid, p, C, ldc, sc, plain, S, Kc, sps, kit, kiv, conj);
}

// Tile and K splits of a dense BF16-term product: the pair of least estimated
// time, from the steps each CU works off (the costs above), about 5 us of
// launch, first loads and stores, and for a split the reduction's launch and
// its pass over the partial products (about 3 TB/s).  Splits keep at least two
// K steps each.
template <int TERMS>
double choose_split_tile(int M, int N, int K, int batch, size_t ws_bytes, int* tile, int* S) {
  using TS = SplitTiles<TERMS>;
  const double mn = (double)M * N * sizeof(float2);
  double best = 0.0;
  *tile = TS::n - 1;
  *S = 1;
  for (int t = 0; t < TS::n; ++t) {
    const TileCost& c = TS::cost[t];
    const double tiles = (double)((M + c.tm - 1) / c.tm) * ((N + c.tn - 1) / c.tn) * batch;
    for (int q : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
      if (q > 1 && (batch != 1 || K < 2 * BKS * q || q * mn > (double)ws_bytes)) break;
      const double steps = std::ceil(std::ceil((double)K / q) / BKS), per_cu = std::ceil(tiles * q / 256.0);
      double us = 5.0 + steps * (per_cu > 1.0 ? std::max(c.alone, per_cu * c.shared) : c.alone);
      if (q > 1) us += 4.0 + (2 * q + 1) * mn / 3e6;
      if (best == 0.0 || us < best) {
        best = us;
        *tile = t;
        *S = q;
      }
    }
  }
  return best;
}

// Tiles of the products on term images, as TileCost (14000 x 2048 x 1021, 4096
// x 2048 x 1021, 1500 x 1000 x 3500, 1000 x 500 x 1000; TERMS 1, largest to
// smallest tile: 196, 63, 70, 21 us and 258, 75, 72, 17; TERMS 2 10752 x 1402 x
// 768 / 701 x 11917 x 1536: 218 / 277 us, 128 x 64: 220 / 286).
template <int TERMS> struct ImageTiles;
template <> struct ImageTiles<1> {
  static constexpr int n = 2;
  static constexpr TileCost cost[n] = {{128, 64, 0.6, 0.44}, {64, 64, 0.4, 0.28}};
  using T0 = ImageTile<1, 128, 64, 2, 2, 2, 3>;
  using T1 = ImageTile<1, 64, 64, 2, 2, 1, 4>;
};
template <> struct ImageTiles<2> {
  static constexpr int n = 1;
  static constexpr TileCost cost[n] = {{64, 64, 0.75, 0.59}};
  using T0 = ImageTile<2, 64, 64, 2, 2, 1, 4>;
  using T1 = T0;
};

// How a product on images is cut so that they fit the scratch: slabs of M, of N
// or of K (then C is read and written again by each).
struct ImagePlan {
  int tile, S, ms, ns, ks;   // tile of ImageTiles; K splits; rows, columns and k of a slab
  double us;
};

inline long long ceil_to(long long a, long long b) { return (a + b - 1) / b * b; }

// bytes of the image of `rows` rows and k numbers, rows padded to whole tiles
template <int TERMS> long long image_bytes(long long rows, long long k, int tile) {
  return ceil_to(rows, tile) * ceil_to(k, BKS) * 2 * TERMS * (long long)sizeof(short);
}

// The cut of least estimated time, from the steps each CU works off as above
// and a conversion of 3.5 us and 5 TB/s; us < 0: none fits.
template <int TERMS>
ImagePlan choose_images(int M, int N, int K, size_t ws_bytes) {
  using TS = ImageTiles<TERMS>;
  ImagePlan best{0, 1, M, N, K, -1.0};
  if (std::max(M, N) > 65535 * IROWS) return best;   // the conversion's grid
  const double mn = (double)M * N * sizeof(float2);
  for (int t = 0; t < TS::n; ++t) {
    const TileCost& c = TS::cost[t];
    const int nt = (N + c.tn - 1) / c.tn, mt = (M + c.tm - 1) / c.tm;
    auto gemm_us = [&](int rows, int cols, int k, int S) {   // rows and columns of tiles
      const double per_cu = std::ceil((double)rows * cols * S / 256.0);
      const double steps = std::ceil(std::ceil((double)k / S) / BKS);
      return 4.0 + steps * (per_cu > 1.0 ? std::max(c.alone, per_cu * c.shared) : c.alone);
    };
    auto convert_us = [&](double rows, double k) { return 3.5 + rows * k * (8.0 + 4.0 * TERMS) / 5e6; };
    auto consider = [&](int S, int ms, int ns, int ks, double us) {
      if (best.us < 0.0 || us < best.us) best = ImagePlan{t, S, ms, ns, ks, us};
    };
    const double convert = convert_us(M, K) + convert_us(N, K);
    // slabs of rows (columns): the other operand's image and one slab's
    for (int side = 0; side < 2; ++side) {
      const int cut = side ? nt : mt, whole = side ? mt : nt, edge = side ? c.tn : c.tm;
      const long long other = image_bytes<TERMS>(side ? M : N, K, side ? c.tm : c.tn);
      const long long one = image_bytes<TERMS>(edge, K, edge);
      if (other + one > (long long)ws_bytes) continue;
      const int fit = (int)std::min<long long>(cut, ((long long)ws_bytes - other) / one);
      for (int slabs = (cut + fit - 1) / fit; slabs <= cut && slabs <= 16; ++slabs)
        for (int fill = 0; fill < 2; ++fill) {   // even slabs, or such as fill the CUs evenly
          int w = (cut + slabs - 1) / slabs;
          const int unit = 256 / std::gcd(256, whole);
          if (fill) w = std::min(fit, (w + unit - 1) / unit * unit);
          const int n = (cut + w - 1) / w, last = cut - (n - 1) * w;
          consider(1, side ? M : w * edge, side ? w * edge : N, K,
                   convert + 3.5 * (n - 1) + (n - 1) * gemm_us(w, whole, K, 1) + gemm_us(last, whole, K, 1));
        }
    }
    // slabs of k, with or without K splits: both images' slabs and the partial products
    for (int S : {1, 2, 3, 4, 6, 8}) {
      if (K < 4 * BKS * S) break;
      const long long part = S > 1 ? (long long)S * (long long)mn : 0;
      const long long k_img = image_bytes<TERMS>(M, BKS, c.tm) + image_bytes<TERMS>(N, BKS, c.tn);
      const long long kc = ((long long)ws_bytes - part) / k_img;   // k blocks that fit
      if (kc < 4 * S) continue;
      const int n = (int)(((K + BKS - 1) / BKS + kc - 1) / kc);
      const int ks = (int)ceil_to((K + n - 1) / n, BKS);
      double us = convert + 7.0 * (n - 1) + n * gemm_us(mt, nt, ks, S) + (n - 1) * 2 * mn / 3e6;
      if (S > 1) us += n * (4.0 + (2 * S + 1) * mn / 3e6);
      consider(S, M, N, ks, us);
    }
  }
  return best;
}

template <int TERMS>
void launch_images(const Product<float>& p, bool ta, bool tb, int conj, const ImagePlan& g) {
  using TS = ImageTiles<TERMS>;
  const TileCost& c = TS::cost[g.tile];
  const long long mn = (long long)p.M * p.N;
  auto convert = [&](bool kc, const float* X, long long ld, int R, int K, int pad, int cj, unsigned short* img) {
    const dim3 grid((K + BKS - 1) / BKS, (unsigned)(ceil_to(R, pad) / IROWS));
    if (kc) hipLaunchKernelGGL((terms_kernel<true, TERMS>), grid, dim3(256), 0, p.s, X, ld, R, K, cj, img);
    else hipLaunchKernelGGL((terms_kernel<false, TERMS>), grid, dim3(256), 0, p.s, X, ld, R, K, cj, img);
  };
  for (long long k0 = 0; k0 < p.K; k0 += g.ks) {
    const int K = (int)std::min<long long>(g.ks, p.K - k0), nkc = (K + BKS - 1) / BKS;
    const int Kc = (int)ceil_to((K + g.S - 1) / g.S, BKS), S = (K + Kc - 1) / Kc;
    unsigned short* ia = static_cast<unsigned short*>(p.ws);
    unsigned short* ib = ia + image_bytes<TERMS>(g.ms, K, c.tm) / 2;
    float* part = reinterpret_cast<float*>(ib + image_bytes<TERMS>(g.ns, K, c.tn) / 2);
    const float br = k0 ? 1.f : p.br, bi = k0 ? 0.f : p.bi;
    // rows m0 .. of A, columns n0 .. of B; at most one of the two is cut
    auto a_rows = [&](long long m0, int M) {
      convert(!ta, p.A + 2 * (ta ? k0 * p.lda + m0 : m0 * p.lda + k0), p.lda, M, K, c.tm, conj & 1, ia);
    };
    if (g.ms >= p.M) a_rows(0, p.M);
    for (long long n0 = 0; n0 < p.N; n0 += g.ns) {
      const int N = (int)std::min<long long>(g.ns, p.N - n0);
      convert(tb, p.B + 2 * (tb ? n0 * p.ldb + k0 : k0 * p.ldb + n0), p.ldb, N, K, c.tn, conj & 2, ib);
      for (long long m0 = 0; m0 < p.M; m0 += g.ms) {
        const int M = (int)std::min<long long>(g.ms, p.M - m0);
        if (g.ms < p.M) a_rows(m0, M);
        const dim3 grid((N + c.tn - 1) / c.tn, (M + c.tm - 1) / c.tm, S);
        float* C = p.C + 2 * (m0 * p.ldc + n0);
        auto product = [&](auto tl) {
          using TL = decltype(tl);
          auto go = [&](auto beta, float alr, float ali, float* out, long long ldo, int parts, long long sps) {
            hipLaunchKernelGGL((gemm_image_kernel<TL, decltype(beta)::value>), grid, dim3(TL::NTH), 0, p.s, M, N, K, alr,
                               ali, ia, ib, nkc, br, bi, out, ldo, parts, Kc, sps);
          };
          if (S > 1) go(std::false_type{}, 1.f, 0.f, part, N, S, mn);
          else if (br == 0.f && bi == 0.f) go(std::false_type{}, p.ar, p.ai, C, p.ldc, 1, 0);
          else go(std::true_type{}, p.ar, p.ai, C, p.ldc, 1, 0);
        };
        if (g.tile == 0) product(typename TS::T0{});
        else product(typename TS::T1{});
        if (S > 1)
          hipLaunchKernelGGL(splitk_reduce_kernel<float>, dim3((unsigned)((mn + 255) / 256)), dim3(256), 0, p.s, part, S,
                             (long long)M, (long long)N, p.ar, p.ai, br, bi, C, p.ldc);
      }
    }
  }
}

// Number of K splits of an FP64 product: about one 64 x 64 tile per CU when the
// output has few (Gram matrices, back transformations), each keeping >= 64 of
// K.  ws_bytes: room for the partial products.
inline int choose_splits(int M, int N, int K, int batch, size_t ws_bytes) {
  const long long tiles = (long long)((M + BM - 1) / BM) * ((N + BN - 1) / BN) * batch;
  if (batch != 1 || ws_bytes == 0 || tiles >= 256 || K < 128) return 1;
  int S = (int)std::min<long long>((256 + tiles - 1) / tiles, K / 64);
  S = std::min(S, 32);
  while (S > 1 && (size_t)S * M * N * sizeof(double2) > ws_bytes) --S;
  return std::max(S, 1);
}

using Direct0 = DirectTile<2, 2, 2, 2, 1, 6>;
using Direct1 = DirectTile<2, 1, 2, 2, 1, 4>;
using Direct2 = DirectTile<1, 1, 2, 2, 1, 8>;
using Direct3 = DirectTile<2, 2, 1, 1, 8, 4>;
using Direct4 = DirectTile<2, 1, 1, 1, 8, 4>;
using Direct5 = DirectTile<1, 1, 1, 1, 16, 8>;
using DirectMapped = DirectTile<2, 2, 2, 2, 1, 4, true>;
using DirectWide = DirectTile<2, 2, 2, 2, 1, 2, true, true>;
constexpr int N_DIRECT = 6;

// Estimated time in us of an M x N x K product in S parts on a tile (infinite
// where the tile takes no such parts), from what the busiest CU works off: 80
// ns a piece and step on each SIMD, and the operand loads.  These cost 6 us a
// MiB and CU where k is not the contiguous index, 10 where it is (a load meets
// 16 rows), 16 where it is for both operands; half as much again with one wave
// a SIMD (not in the last case), 0.6 of it in pieces of 32 x 32.  Blocks of two
// or three waves land unevenly on the SIMDs.  A second launch sums the partial
// products of a split grid.
template <class TL, bool TA, bool TB> double direct_cost(int M, int N, int K, int batch, int S, bool in_block) {
  if (in_block ? S > TL::PARTS : S > 1 && TL::PARTS > 1) return 1e30;
  const double mn = (double)M * N * sizeof(double2);
  const double blocks = (double)((M + TL::TM - 1) / TL::TM) * ((N + TL::TN - 1) / TL::TN) * (in_block ? 1 : S) * batch;
  const double per_cu = std::ceil(blocks / 256.0), waves = TL::WM * TL::WN * (in_block ? S : 1);
  // a CU holds eight blocks of one 32 x 32 wave, and one to four after a full round
  // run at the pace of a lone wave: 474 x 5086 x 198 (ten a CU) 91 us, four waves a block
  // 69 (64 x 64 tiles through LDS 72), 2235 x 966 x 371 152 / 118 (128); over random
  // shapes of 9 to 12, 17 to 20 and 25 to 28 a CU 1.10 to 1.12 times the time, of 13 to
  // 16 and 37 to 40 0.99 to 1.01 (3148 x 1307 x 104 61 / 71)
  if (S == 1 && TL::PARTS > 1 && TL::SI * TL::SJ == 4 && per_cu > 8.0 && (int)(per_cu - 1.0) % 8 < 4) return 1e30;
  const double steps = std::ceil(std::ceil((double)K / S) / 4);
  double per_simd = std::ceil(per_cu * waves / 4.0);
  if (waves == 2.0 || waves == 3.0) per_simd = std::max(per_simd, 2.0);
  const double mib = per_cu * waves * steps / 1024.0;
  constexpr bool both = !TA && TB;
  constexpr double wa = both ? 16.0 : TA ? 6.0 : 10.0, wb = both ? 16.0 : TB ? 10.0 : 6.0;
  const double load = mib * (TL::SI * wa + TL::SJ * wb) * (TL::SI * TL::SJ == 4 ? 0.6 : 1.0) *
                      (per_simd > 1.0 || both ? 1.0 : 1.5);
  double us = 4.5 + per_simd * steps * TL::SI * TL::SJ * 0.08 + load;
  if (S > 1) us += in_block ? per_cu * 0.03 * S * TL::SI * TL::SJ : 4.0 + (2 * S + 1) * mn / 8e6;
  return us;
}

// Tile of a dense FP64 product of S parts: the least estimated time, from what
// the busiest CU works off.  Large outputs take the 64 x 64 tile (fewest
// operand bytes per output); smaller ones take smaller tiles, which fill more
// of the 256 CUs, with the parts of K on a block's waves instead of a second
// launch.  Measured with 64 x 64 tiles through LDS / on these tiles: 256 x 64 x
// 32 7.5 / 3.7 us, 64 x 32 x 256 14.1 / 5.4, 768 x 192 x 96 15.5 / 7.0, 192 x
// 96 x 768 17.2 / 11, 462 x 256 x 256 18.4 / 8.4, 512 x 256 x 2048 43.5 / 38.8,
// 2048 x 512 x 256 37.3 / 34.3, 5000 x 1000 x 1000 652 / 511.
template <bool TA, bool TB>
void choose_direct_tile(int M, int N, int K, int batch, int S, int* tile, bool* in_block) {
  double best = 1e29;
  *tile = 0;
  *in_block = false;
  // Few steps and many outputs: what counts is how many waves a SIMD holds (four of
  // tile 1, two of tiles 0 and 3), on the largest products the loads too, and whole
  // lines of C where its rows are short.  Tile 0 / 1 / by the estimate / 64 x 64 tiles
  // through LDS in us: 1537 x 1679 x 25 20.1 / 18.2 / 23.8 / 21.2, 1598 x 2987 x 22
  // 27 / 23 / 29.5 / 30, 3500 x 3500 x 20 52 / 45 / - / 59, 5912 x 3503 x 21 102 / 114 /
  // 103 / 112, 295595 x 45 x 18 with beta 118 / 151 / 135 / 114.  Rows of C of two
  // tiles of 32 lose their lines only where the two run on different XCDs, not where
  // the tiles are dealt in bands (a multiple of eight, see tile_job), with beta: 5219 x
  // 56 x 12 (30) 51.3 / 48.8 / - / 50, 102400 x 50 x 30 50 / 40 / - / 48; 6250 tiles of
  // 200000 x 45 x 12 56 / 68 / - / 54; nor past the 256 MB memory-side cache, 204800 x
  // 60 x 30 112 / 119 / - / 103.
  const double mn = (double)M * N * batch;
  if (S == 1 && K <= 32 && mn >= 1e6) {
    const long long tiles = (long long)((M + Direct1::TM - 1) / Direct1::TM) * ((N + Direct1::TN - 1) / Direct1::TN) * batch;
    const double bytes = (mn + ((double)M + N) * K * batch) * sizeof(double2);
    const bool bands = tiles % 8 == 0 && bytes <= 256e6;
    *tile = (mn <= 1.8e7 || mn * K <= 2.5e8) && (N <= 32 || N >= 64 || bands) ? 1 : 0;
    return;
  }
  for (int ib = 0; ib < 2; ++ib) {
    if (ib && S == 1) break;
    const double us[N_DIRECT] = {
        direct_cost<Direct0, TA, TB>(M, N, K, batch, S, ib), direct_cost<Direct1, TA, TB>(M, N, K, batch, S, ib),
        direct_cost<Direct2, TA, TB>(M, N, K, batch, S, ib), direct_cost<Direct3, TA, TB>(M, N, K, batch, S, ib),
        direct_cost<Direct4, TA, TB>(M, N, K, batch, S, ib), direct_cost<Direct5, TA, TB>(M, N, K, batch, S, ib)};
    for (int t = 0; t < N_DIRECT; ++t)
      if (us[t] < best) {
        best = us[t];
        *tile = t;
        *in_block = ib != 0;
      }
  }
}

// parts > 1: K in parts of Kc on the block's waves
template <class TL, bool TA, bool TB, int TAG>
void launch_direct_tile(const Product<double>& p, int n_items, double* C, long long ldc, long long sc, bool plain,
                        int S, int parts, int Kc, long long sps, const int4* kit, const int2* kiv, int conj) {
  const dim3 grid = kit ? dim3(n_items)
                        : dim3((p.N + TL::TN - 1) / TL::TN, (p.M + TL::TM - 1) / TL::TM, S > 1 ? S : p.batch);
  const size_t lds = parts > 1 ? (size_t)parts * TL::SI * TL::SJ * 256 * sizeof(double2) : 0;
  auto go = [&](auto beta) {
    const auto kernel = gemm_direct_kernel<TL, TA, TB, decltype(beta)::value, TAG>;
    if (lds > 64 * 1024) {   // per device, and cheap next to a launch that takes this much
      HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    }
    hipLaunchKernelGGL(kernel, grid, dim3(TL::WM * TL::WN * parts * 64), lds, p.s, p.M, p.N, p.K, plain ? 1.0 : p.ar,
                       plain ? 0.0 : p.ai, p.A, p.lda, p.sa, p.B, p.ldb, p.sb, plain ? 0.0 : p.br,
                       plain ? 0.0 : p.bi, C, ldc, sc, S, Kc, sps, kit, kiv, conj);
  };
  if (plain || (p.br == 0.0 && p.bi == 0.0)) go(std::false_type{});
  else go(std::true_type{});
}

template <bool TA, bool TB, int TAG>
void launch_direct(const Product<double>& p, int conj, int tile, int n_items, double* C, long long ldc, long long sc,
                   bool plain, int S, int parts, int Kc, long long sps, const int4* kit, const int2* kiv) {
  auto go = [&](auto tl) {
    launch_direct_tile<decltype(tl), TA, TB, TAG>(p, n_items, C, ldc, sc, plain, S, parts, Kc, sps, kit, kiv, conj);
  };
  if (wide_ld(p.lda, p.ldb, LD_WIDE64)) return go(DirectWide{});
  if (kit) return go(DirectMapped{});
  switch (tile) {
    case 0: return go(Direct0{});
    case 1: return go(Direct1{});
    case 2: return go(Direct2{});
    case 3: return go(Direct3{});
    case 4: return go(Direct4{});
    default: return go(Direct5{});
  }
}

// TERMS 0: FP64; otherwise complex64 operands as TERMS BF16 terms.
template <typename T, int TERMS, int OA, int OB, int TAG>
void launch_gemm_mode(const Product<T>& p) {
  constexpr bool TA = (OA == TDVP_OP_T || OA == TDVP_OP_C), CA = (OA == TDVP_OP_C || OA == TDVP_OP_R);
  constexpr bool TB = (OB == TDVP_OP_T || OB == TDVP_OP_C), CB = (OB == TDVP_OP_C || OB == TDVP_OP_R);
  constexpr int KSTEP = TERMS == 0 ? 16 : BKS, CONJ = (CA ? 1 : 0) | (CB ? 2 : 0);
  using c2 = typename VT<T>::c2;
  const int M = p.M, N = p.N, K = p.K, batch = p.batch;
  const long long MN = (long long)M * N;
  // S > 1 or `plain`: partial products (alpha 1, beta 0)
  auto launch = [&](int tile, int n_items, T* C, long long ldc, long long sc, bool plain, int S, int Kc, long long sps,
                    const int4* kit, const int* kiv, int parts = 1) {
    const int2* iv = reinterpret_cast<const int2*>(kiv);
    if constexpr (TERMS == 0)
      launch_direct<TA, TB, TAG>(p, CONJ, tile, n_items, C, ldc, sc, plain, S, parts, Kc, sps, kit, iv);
    else
      launch_split<TERMS, TA, TB, TAG>(p, CONJ, tile, n_items, C, ldc, sc, plain, S, Kc, sps, kit, iv);
  };
  const kern::KMap* km = tl_kmap;
  if (km && km->batch == batch) {
    if (km->M != M || km->N != N || km->K != K) TDVP_THROW(TDVP_ERR_ARG, "block-sparse map does not fit the product");
    const int gx = (N + BN - 1) / BN;
    if (km->splits > 1) {
      if (!km->part || km->part_bytes < (size_t)km->splits * batch * MN * sizeof(c2))
        TDVP_THROW(TDVP_ERR_ARG, "block-sparse map without room for its partial products");
      T* P = static_cast<T*>(km->part);
      if (km->n_items > 0)
        launch(0, km->n_items, P, N, MN, true, km->splits, std::max(K, 1), MN * batch, km->items, km->iv);
      hipLaunchKernelGGL(splitk_reduce_map_kernel<T>, dim3((unsigned)((MN * batch + 255) / 256)), dim3(256), 0, p.s, P,
                         batch, (long long)M, (long long)N, gx, km->tinfo, p.ar, p.ai, p.br, p.bi, p.C, p.ldc, p.sc);
      return;
    }
    if (!km->partial && km->n_items < batch * gx * ((M + BM - 1) / BM))
      TDVP_THROW(TDVP_ERR_ARG, "block-sparse map without every tile");
    if (km->n_items == 0) return;   // a partial map with nothing to write
    launch(0, km->n_items, p.C, p.ldc, p.sc, false, 1, std::max(K, 1), 0, km->items, km->iv);
    return;
  }
  int S, tile = 0;
  bool in_block = false;
  if constexpr (TERMS == 0) {
    S = choose_splits(M, N, K, batch, p.ws_bytes);
    choose_direct_tile<TA, TB>(M, N, K, batch, S, &tile, &in_block);
    if (wide_ld(p.lda, p.ldb, LD_WIDE64)) in_block = false;
  } else {
    if constexpr (TERMS == 3) {
      if (short_product(p)) {
        launch_short<TA, TB>(p, CONJ);
        return;
      }
    }
    const double us = choose_split_tile<TERMS>(M, N, K, batch, p.ws_bytes, &tile, &S);
    // on term images where those take less time: large products, and long ones
    // whose few tiles repeat the conversion one after the other
    if constexpr (TERMS < 3) {
      Product<float> q = p;
      const size_t skip = (256 - reinterpret_cast<uintptr_t>(p.ws) % 256) % 256;
      if (batch == 1 && K > 0 && p.ws && p.ws_bytes > skip) {
        q.ws = static_cast<char*>(p.ws) + skip;
        q.ws_bytes -= skip;
        const ImagePlan g = choose_images<TERMS>(M, N, K, q.ws_bytes);
        if (g.us > 0.0 && g.us < us) {
          launch_images<TERMS>(q, TA, TB, CONJ, g);
          return;
        }
      }
    }
  }
  if (S == 1) {
    launch(tile, 0, p.C, p.ldc, p.sc, false, 1, std::max(K, 1), 0, nullptr, nullptr);
    return;
  }
  const int Kc = ((K + S - 1) / S + KSTEP - 1) / KSTEP * KSTEP;
  const int Sx = (K + Kc - 1) / Kc;
  if (in_block) {
    launch(tile, 0, p.C, p.ldc, p.sc, false, 1, Kc, 0, nullptr, nullptr, Sx);
    return;
  }
  T* P = static_cast<T*>(p.ws);
  launch(tile, 0, P, N, 0, true, Sx, Kc, MN, nullptr, nullptr);
  hipLaunchKernelGGL(splitk_reduce_kernel<T>, dim3((unsigned)((MN + 255) / 256)), dim3(256), 0, p.s, P, Sx,
                     (long long)M, (long long)N, p.ar, p.ai, p.br, p.bi, p.C, p.ldc);
}

template <typename T, int OA, int OB, int TAG = 0>
void launch_gemm(hipStream_t s, int M, int N, int K, zc alpha, const void* A, long long lda,
                 long long sa, const void* B, long long ldb, long long sb, zc beta, void* C,
                 long long ldc, long long sc, int batch, void* ws = nullptr, size_t ws_bytes = 0) {
  const Product<T> p{s, M, N, K, batch, static_cast<const T*>(A), lda, sa, static_cast<const T*>(B), ldb, sb,
                     static_cast<T*>(C), ldc, sc, T(alpha.real()), T(alpha.imag()), T(beta.real()), T(beta.imag()),
                     ws, ws ? ws_bytes : 0};
  if constexpr (sizeof(T) == 8) {
    launch_gemm_mode<T, 0, OA, OB, TAG>(p);
  } else {
    if (tl_float_mode == 1) launch_gemm_mode<T, 1, OA, OB, TAG>(p);
    else if (tl_float_mode == 2) launch_gemm_mode<T, 2, OA, OB, TAG>(p);
    else launch_gemm_mode<T, 3, OA, OB, TAG>(p);
  }
}

template <typename T, int OA>
void dispatch_b(hipStream_t s, int opb, int M, int N, int K, zc alpha, const void* A, long long lda,
                long long sa, const void* B, long long ldb, long long sb, zc beta, void* C,
                long long ldc, long long sc, int batch, void* ws, size_t wsb) {
  switch (opb) {
    case TDVP_OP_N: launch_gemm<T, OA, TDVP_OP_N>(s, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, wsb); break;
    case TDVP_OP_T: launch_gemm<T, OA, TDVP_OP_T>(s, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, wsb); break;
    case TDVP_OP_C: launch_gemm<T, OA, TDVP_OP_C>(s, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, wsb); break;
    case TDVP_OP_R: launch_gemm<T, OA, TDVP_OP_R>(s, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, wsb); break;
    default: TDVP_THROW(TDVP_ERR_ARG, "bad GEMM op_b");
  }
}

// ---------------------------------------------------------------- W apply
// Memory bound.  An MPO tensor holds about one nonzero per input channel, so an
// input entry is read once or twice: each wave takes output channels of one row
// p and 64 V columns (V entries a lane, 16 bytes) and reads its inputs straight
// from memory, the coefficients through scalar loads.
// chi = 1024, w = 20, complex64, dense: 108 us, 6.2 TB/s (through LDS, eight
// bytes a lane: 184 us).
constexpr int WNT = 256;

// the MPO tensor in device memory; kern::WInline: in the kernel's arguments
struct WPointers {
  const int* __restrict__ rowptr;
  const int* __restrict__ col;
  const double* __restrict__ val;
};

template <typename T, int V, bool CHARGED, class TAB>
__global__ __launch_bounds__(WNT) void wapply_kernel(const T* __restrict__ in, T* __restrict__ out, long long nQ,
                                                      long long isP, long long is1, long long is2, long long osP,
                                                      long long os1, long long os2, const TAB tab, int n_out,
                                                      kern::WCharges wc) {
  using c2 = typename VT<T>::c2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long p = blockIdx.y;
  const long long q = ((long long)blockIdx.x * 64 + (threadIdx.x & 63)) * V;
  if (q >= nQ) return;
  const c2* inb = reinterpret_cast<const c2*>(in) + p * isP + q;
  c2* outb = reinterpret_cast<c2*>(out) + p * osP + q;
  const bool whole = q + V <= nQ;
  // charge difference of the lane's columns (charged contractions only); an
  // output of another charge is an exact zero, stored unless the output already
  // holds it, and an output's inputs all have its charge
  int dq[V];
  if constexpr (CHARGED) {
    const int ql = wc.ql[p];
#pragma unroll
    for (int v = 0; v < V; ++v) dq[v] = wc.qr[q + v < nQ ? q + v : q] - ql;
  }
  for (int o = blockIdx.z * (WNT / 64) + wave; o < n_out; o += gridDim.z * (WNT / 64)) {
    bool on[V], any = false, all = whole;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      on[v] = (V == 1 || v == 0 || whole) && (!CHARGED || wc.dout[o] == dq[v]);
      any = any || on[v];
      all = all && on[v];
    }
    T sr[V], si[V];
#pragma unroll
    for (int v = 0; v < V; ++v) sr[v] = si[v] = T(0);
    if (any) {
      const int e1 = tab.rowptr[o + 1];
      for (int e = tab.rowptr[o]; e < e1; ++e) {
        const double2 w = make_double2(tab.val[2 * e], tab.val[2 * e + 1]);
        const int c = tab.col[e];
        const c2* x = inb + (c >> 1) * is1 + (c & 1) * is2;
        c2 xv[V];
        if constexpr (V == 2) {
          if (whole) {
            const f4u t = *reinterpret_cast<const f4u*>(x);
            xv[0].x = t.x;
            xv[0].y = t.y;
            xv[1].x = t.z;
            xv[1].y = t.w;
          } else {
            xv[0] = xv[1] = x[0];
          }
        } else {
          xv[0] = x[0];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
          sr[v] += T(w.x) * xv[v].x - T(w.y) * xv[v].y;
          si[v] += T(w.x) * xv[v].y + T(w.y) * xv[v].x;
        }
      }
    }
    c2* y = outb + (o >> 1) * os1 + (o & 1) * os2;
    const bool keep = CHARGED && wc.zeros_kept;
    if constexpr (V == 2) {
      if (all || (whole && !keep)) {
        f4u t;
        t.x = on[0] ? sr[0] : T(0);
        t.y = on[0] ? si[0] : T(0);
        t.z = on[1] ? sr[1] : T(0);
        t.w = on[1] ? si[1] : T(0);
        *reinterpret_cast<f4u*>(y) = t;
        continue;
      }
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
      if ((v == 0 || whole) && (on[v] || !keep)) {
        c2 r;
        r.x = on[v] ? sr[v] : T(0);
        r.y = on[v] ? si[v] : T(0);
        y[v] = r;
      }
  }
}

// Tensors with many nonzeros on large operands: a wave takes an output channel
// at a time, and its inputs, 64 columns of a row, pass through LDS (64 KiB for the
// 64 channels of complex128), since waves that read them in different orders read
// past the caches: each comes from memory once here.  The sums are the direct
// kernel's, in its order.  Times of a whole matvec: see wapply_by_lds.
template <typename T, bool CHARGED, class TAB>
__global__ __launch_bounds__(WNT) void wapply_lds_kernel(const T* __restrict__ in, T* __restrict__ out, long long nQ,
                                                          long long isP, long long is1, long long is2, long long osP,
                                                          long long os1, long long os2, const TAB tab, int n_in,
                                                          int n_out, kern::WCharges wc) {
  using c2 = typename VT<T>::c2;
  extern __shared__ __attribute__((aligned(16))) unsigned char wapply_lds[];
  c2* x = reinterpret_cast<c2*>(wapply_lds);   // [channel][column]
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long p = blockIdx.y, q = (long long)blockIdx.x * 64 + lane;
  const bool there = q < nQ;
  const c2* inb = reinterpret_cast<const c2*>(in) + p * isP + q;
  c2* outb = reinterpret_cast<c2*>(out) + p * osP + q;
  const int dq = CHARGED && there ? wc.qr[q] - wc.ql[p] : 0;
  for (int c = wave; c < n_in; c += WNT / 64) {
    c2 v;
    v.x = v.y = T(0);
    if (there && (!CHARGED || wc.din[c] == dq)) v = inb[(c >> 1) * is1 + (c & 1) * is2];
    x[c * 64 + lane] = v;
  }
  __syncthreads();
  if (!there) return;
  for (int o = wave; o < n_out; o += WNT / 64) {
    const bool on = !CHARGED || wc.dout[o] == dq;
    if (!on && wc.zeros_kept) continue;
    T sr = T(0), si = T(0);
    if (on) {
      const int e1 = tab.rowptr[o + 1];
      for (int e = tab.rowptr[o]; e < e1; ++e) {
        const double2 w = make_double2(tab.val[2 * e], tab.val[2 * e + 1]);
        const c2 v = x[tab.col[e] * 64 + lane];
        sr += T(w.x) * v.x - T(w.y) * v.y;
        si += T(w.x) * v.y + T(w.y) * v.x;
      }
    }
    c2 r;
    r.x = sr;
    r.y = si;
    outb[(o >> 1) * os1 + (o & 1) * os2] = r;
  }
}

// ---------------------------------------------------------------- vectors
constexpr int VNT = 256;
constexpr int DOT_CHUNK = 1024;

// sum over the wave (all 64 lanes active; every lane gets the total)
__device__ inline double warp_sum(double v) { return wave::sum(v); }

__device__ inline double block_sum(double v, double* sh) {
  v = warp_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < VNT / 64; ++i) t += sh[i];
  return t;  // valid on thread 0
}

// One block per (vector j, chunk): partial[b * nv + j] = sum over the chunk.
template <bool CONJ>
__global__ __launch_bounds__(VNT) void zdots_partial_kernel(const double2* __restrict__ V, long long ldv, int nv,
                                                             const double2* __restrict__ w, long long n,
                                                             double2* __restrict__ partial) {
  __shared__ double sh[VNT / 64];
  const int j = blockIdx.y;
  const long long beg = (long long)blockIdx.x * DOT_CHUNK;
  const long long end = min(n, beg + DOT_CHUNK);
  double sr = 0.0, si = 0.0;
  const double2* v = V + (long long)j * ldv;
  for (long long x = beg + threadIdx.x; x < end; x += VNT) {
    const double2 a = v[x], b = w[x];
    if (CONJ) {                    // conj(a) * b
      sr += a.x * b.x + a.y * b.y;
      si += a.x * b.y - a.y * b.x;
    } else {                       // a * b
      sr += a.x * b.x - a.y * b.y;
      si += a.x * b.y + a.y * b.x;
    }
  }
  const double tr = block_sum(sr, sh);
  const double ti = block_sum(si, sh);
  if (threadIdx.x == 0) partial[(long long)blockIdx.x * nv + j] = make_double2(tr, ti);
}

// one block per vector: out[j] = sum over the blocks' partials (fixed tree)
__global__ __launch_bounds__(VNT) void zdots_final_kernel(const double2* __restrict__ partial, int nb, int nv,
                                                           double2* __restrict__ out) {
  __shared__ double sh[VNT / 64];
  const int j = blockIdx.x;
  double sr = 0.0, si = 0.0;
  for (int b = threadIdx.x; b < nb; b += VNT) {
    const double2 p = partial[(long long)b * nv + j];
    sr += p.x;
    si += p.y;
  }
  const double tr = block_sum(sr, sh);
  const double ti = block_sum(si, sh);
  if (threadIdx.x == 0) out[j] = make_double2(tr, ti);
}

// dst = V c, the coefficients in the kernel's arguments (a copy, a fill and a
// wait for the copy less: 1.6 ms of a sweep's 34 at chi = 96)
constexpr int ZC_ARGS = 64;
struct CombineArgs {
  double2 c[ZC_ARGS];
};
__global__ __launch_bounds__(VNT) void zcombine_args_kernel(double2* __restrict__ dst, const double2* __restrict__ V,
                                                             long long ldv, int nv, const CombineArgs c, long long n) {
  const long long x = (long long)blockIdx.x * VNT + threadIdx.x;
  if (x >= n) return;
  double sr = 0.0, si = 0.0;
  for (int j = 0; j < nv; ++j) {
    const double2 cj = c.c[j];
    const double2 v = V[(long long)j * ldv + x];
    sr += cj.x * v.x - cj.y * v.y;
    si += cj.x * v.y + cj.y * v.x;
  }
  dst[x] = make_double2(0.0 + sr, 0.0 + si);
}

__global__ void zscale_kernel(double2* __restrict__ dst, const double2* __restrict__ src, double ar,
                              double ai, long long n) {
  const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const double2 v = src[x];
  dst[x] = make_double2(ar * v.x - ai * v.y, ar * v.y + ai * v.x);
}

// w += sign * V c with c_j the sum of the nb partial dot products
// partial[b * nv + j] (zdots_partial_kernel's layout): every block forms c
// itself, in the same fixed order, so no separate reduction launch is
// needed; block 0 also stores c in cout.  With NORM, the block's partial sum
// of |w|^2 goes to npart.
constexpr int ZC_MAXV = 64;
template <bool NORM>
__global__ __launch_bounds__(VNT) void zcombine_p_kernel(double2* __restrict__ w, const double2* __restrict__ V,
                                                         long long ldv, int nv, const double2* __restrict__ partial,
                                                         int nb, double sign, long long n, double2* __restrict__ cout,
                                                         double2* __restrict__ npart) {
  __shared__ double2 sc[ZC_MAXV];
  __shared__ double sh[VNT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int j = wv; j < nv; j += VNT / 64) {
    double re = 0.0, im = 0.0;
    for (int b = lane; b < nb; b += 64) {
      const double2 p = partial[(long long)b * nv + j];
      re += p.x;
      im += p.y;
    }
    re = warp_sum(re);
    im = warp_sum(im);
    if (lane == 0) sc[j] = make_double2(re, im);
  }
  __syncthreads();
  if (blockIdx.x == 0 && cout)
    for (int j = threadIdx.x; j < nv; j += VNT) cout[j] = sc[j];
  const long long x = (long long)blockIdx.x * VNT + threadIdx.x;
  double sq = 0.0;
  if (x < n) {
    double sr = 0.0, si = 0.0;
    for (int j = 0; j < nv; ++j) {
      const double2 cj = sc[j];
      const double2 v = V[(long long)j * ldv + x];
      sr += cj.x * v.x - cj.y * v.y;
      si += cj.x * v.y + cj.y * v.x;
    }
    double2 o = w[x];
    o.x += sign * sr;
    o.y += sign * si;
    w[x] = o;
    sq = o.x * o.x + o.y * o.y;
  }
  if (NORM) {
    const double t = block_sum(sq, sh);
    if (threadIdx.x == 0) npart[blockIdx.x] = make_double2(t, 0.0);
  }
}

// The same update, then the block's partial dot products of the updated w
// with every vector, dpart[blockIdx.x * nv + j] = sum over the block's x of
// conj(V[j][x]) w[x] (the layout zcombine_p_kernel reads): the second
// Gram-Schmidt pass gets its projections without another read of V.
__global__ __launch_bounds__(VNT) void zcombine_dots_kernel(double2* __restrict__ w, const double2* __restrict__ V,
                                                            long long ldv, int nv,
                                                            const double2* __restrict__ partial, int nb,
                                                            double sign, long long n, double2* __restrict__ cout,
                                                            double2* __restrict__ dpart) {
  __shared__ double2 sc[ZC_MAXV];
  __shared__ double2 sd[VNT / 64][ZC_MAXV];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int j = wv; j < nv; j += VNT / 64) {
    double re = 0.0, im = 0.0;
    for (int b = lane; b < nb; b += 64) {
      const double2 p = partial[(long long)b * nv + j];
      re += p.x;
      im += p.y;
    }
    re = warp_sum(re);
    im = warp_sum(im);
    if (lane == 0) sc[j] = make_double2(re, im);
  }
  __syncthreads();
  if (blockIdx.x == 0 && cout)
    for (int j = threadIdx.x; j < nv; j += VNT) cout[j] = sc[j];
  const long long x = (long long)blockIdx.x * VNT + threadIdx.x;
  double2 o = make_double2(0.0, 0.0);
  if (x < n) {
    double sr = 0.0, si = 0.0;
    for (int j = 0; j < nv; ++j) {
      const double2 cj = sc[j];
      const double2 v = V[(long long)j * ldv + x];
      sr += cj.x * v.x - cj.y * v.y;
      si += cj.x * v.y + cj.y * v.x;
    }
    o = w[x];
    o.x += sign * sr;
    o.y += sign * si;
    w[x] = o;
  }
  for (int j = 0; j < nv; ++j) {   // uniform loop: every lane takes part in the sums
    double re = 0.0, im = 0.0;
    if (x < n) {
      const double2 v = V[(long long)j * ldv + x];
      re = v.x * o.x + v.y * o.y;
      im = v.x * o.y - v.y * o.x;
    }
    re = warp_sum(re);
    im = warp_sum(im);
    if (lane == 0) sd[wv][j] = make_double2(re, im);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nv; j += VNT) {
    double2 t = sd[0][j];
#pragma unroll
    for (int q = 1; q < VNT / 64; ++q) {
      t.x += sd[q][j].x;
      t.y += sd[q][j].y;
    }
    dpart[(long long)blockIdx.x * nv + j] = t;
  }
}

// every block sums the np partial norms in the same fixed order, so all
// agree on |w|^2; block 0 also stores it
__global__ __launch_bounds__(VNT) void zscale_invnorm_kernel(double2* __restrict__ w,
                                                              const double2* __restrict__ partial, int np,
                                                              double2* __restrict__ out, long long n,
                                                              double2* host, const double2* __restrict__ coeffs,
                                                              int ncoef, int host_norm_at) {
  __shared__ double sh[VNT / 64];
  __shared__ double s_tot;
  double acc = 0.0;
  for (int b = threadIdx.x; b < np; b += VNT) acc += partial[b].x;
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) {
    s_tot = t;
    if (blockIdx.x == 0) {
      out[0] = make_double2(t, 0.0);
      if (host) host[host_norm_at] = make_double2(t, 0.0);
    }
  }
  if (blockIdx.x == 0 && host)
    for (int j = threadIdx.x; j < ncoef; j += VNT) host[j] = coeffs[j];
  __syncthreads();
  const long long x = (long long)blockIdx.x * VNT + threadIdx.x;
  if (x >= n) return;
  const double inv = 1.0 / sqrt(fmax(s_tot, 0.0));
  const double2 v = w[x];
  w[x] = make_double2(v.x * inv, v.y * inv);
}

__global__ void z2c_kernel(float2* __restrict__ dst, const double2* __restrict__ src, long long n) {
  const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const double2 v = src[x];
  dst[x] = make_float2(float(v.x), float(v.y));
}

__global__ void c2z_kernel(double2* __restrict__ dst, const float2* __restrict__ src, long long n) {
  const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const float2 v = src[x];
  dst[x] = make_double2(double(v.x), double(v.y));
}

template <typename E>
__global__ void copy2d_kernel(E* __restrict__ dst, long long ldd, const E* __restrict__ src, long long lds,
                              long long rows, long long cols) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const long long i = idx / cols, j = idx % cols;
  dst[i * ldd + j] = src[i * lds + j];
}

__global__ void ztri_kernel(double2* __restrict__ dst, long long ldd, const double2* __restrict__ src,
                            long long lds, long long rows, long long cols, int mode) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const long long i = idx / cols, j = idx % cols;
  const bool keep = mode == 0 ? (j >= i) : (j <= i);
  dst[i * ldd + j] = keep ? src[i * lds + j] : make_double2(0.0, 0.0);
}

__global__ void zconjtrans_kernel(double2* __restrict__ dst, long long ldd, const double2* __restrict__ src,
                                  long long lds, long long rows, long long cols) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const long long i = idx / cols, j = idx % cols;
  const double2 v = src[j * lds + i];
  dst[i * ldd + j] = make_double2(v.x, -v.y);
}

// A = (S + S^H) / 2 (A may be S: each pair (i, j), j >= i, belongs to one
// thread); thread 0 also clears zero[0 .. nzero)
__global__ void zhermitize_kernel(double2* A, const double2* S, long long n, int* zero, int nzero) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx == 0)
    for (int k = 0; k < nzero; ++k) zero[k] = 0;
  if (idx >= n * n) return;
  const long long i = idx / n, j = idx % n;
  if (j < i) return;
  const double2 a = S[i * n + j], b = S[j * n + i];
  if (i == j) {
    A[i * n + j] = make_double2(a.x, 0.0);
  } else {
    const double2 h = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
    A[i * n + j] = h;
    A[j * n + i] = make_double2(h.x, -h.y);
  }
}

template <typename E>
__global__ void fill_kernel(E* __restrict__ dst, E v, long long n) {
  const long long x = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (x < n) dst[x] = v;
}

__global__ void zscale_phys_kernel(double2* __restrict__ G, long long nx, long long nq, double f0,
                                   double f1) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nx * 2 * nq) return;
  const long long s = (idx / nq) & 1;
  const double f = s ? f1 : f0;
  double2 v = G[idx];
  v.x *= f;
  v.y *= f;
  G[idx] = v;
}

__global__ void zscale_rc_kernel(double2* __restrict__ dst, long long ldd, const double2* __restrict__ src,
                                 long long lds, long long rows, long long cols, const double* __restrict__ f,
                                 int by_col) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= rows * cols) return;
  const long long i = idx / cols, j = idx % cols;
  const double g = by_col ? f[j] : f[i];
  const double2 v = src[i * lds + j];
  dst[i * ldd + j] = make_double2(g * v.x, g * v.y);
}

__global__ void zshift_diag_kernel(double2* __restrict__ G, long long n, double a, double b) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * n) return;
  double2 v = G[idx];
  v.x *= a;
  v.y *= a;
  if (idx / n == idx % n) v.x += b;
  G[idx] = v;
}

// dst[i*ldd + j] = src[r(i)*lds + c(j)], r(i) = ridx ? ridx[i] : i, c likewise
__global__ void zgather_kernel(double2* __restrict__ dst, long long ldd, const double2* __restrict__ src,
                               long long lds, const int* __restrict__ ridx, long long nr,
                               const int* __restrict__ cidx, long long nc) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nr * nc) return;
  const long long i = idx / nc, j = idx % nc;
  const long long r = ridx ? ridx[i] : i, c = cidx ? cidx[j] : j;
  dst[i * ldd + j] = src[r * lds + c];
}

// dst[r(i)*ldd + c(j)] = src[i*lds + j], r(i) = ridx ? ridx[i] : i, c likewise
__global__ void zscatter_kernel(double2* __restrict__ dst, long long ldd, const double2* __restrict__ src,
                                long long lds, const int* __restrict__ ridx, long long nr,
                                const int* __restrict__ cidx, long long nc) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nr * nc) return;
  const long long i = idx / nc, j = idx % nc;
  const long long r = ridx ? ridx[i] : i, c = cidx ? cidx[j] : j;
  dst[r * ldd + c] = src[i * lds + j];
}

template <typename D, typename S>
__device__ inline D cconv(S v) {
  D d;
  d.x = v.x;
  d.y = v.y;
  return d;
}
// block (x, r): entries x * 256 + t of row segment r
template <typename P, typename Dn, bool PACK>
__global__ void rows_pack_kernel(P* __restrict__ packed, Dn* __restrict__ dense, int rows, long long ld,
                                 const int* __restrict__ seg) {
  const int r = blockIdx.y;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int b0 = seg[r], len = seg[rows + r], off = seg[2 * rows + r];
  if (j >= len) return;
  if (PACK) packed[(long long)off + j] = cconv<P>(dense[(long long)r * ld + b0 + j]);
  else dense[(long long)r * ld + b0 + j] = cconv<Dn>(packed[(long long)off + j]);
}

// splitmix64 (Steele, Lea and Flood 2014) as a counter-based generator
__device__ inline unsigned long long mix64(unsigned long long z) {
  z += 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}
__global__ void zrandom_blocks_kernel(double2* __restrict__ E, int R, int C, const int* __restrict__ qr,
                                      const int* __restrict__ qc, unsigned long long seed) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long long)R * C) return;
  const int i = (int)(idx / C), j = (int)(idx % C);
  double2 v{0.0, 0.0};
  if (qr[i] == qc[j]) {
    const unsigned long long a = mix64(seed ^ (2ull * (unsigned long long)idx)),
                             b = mix64(seed ^ (2ull * (unsigned long long)idx + 1ull));
    v.x = (double)(a >> 11) * 0x1.0p-52 - 1.0;
    v.y = (double)(b >> 11) * 0x1.0p-52 - 1.0;
  }
  E[idx] = v;
}

// dst[j] = H[idx[j]*n + idx[j]]; rows[pos[j]*n + idx[j]] = 1 (unit eigenvector of a 1 x 1 block)
__global__ void zunit_blocks_kernel(double2* __restrict__ dst, const double2* __restrict__ H, long long n,
                                    const int* __restrict__ idx, const int* __restrict__ pos, int cnt,
                                    double2* __restrict__ rows) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= cnt) return;
  const long long i = idx[j];
  dst[j] = H[i * n + i];
  rows[(long long)pos[j] * n + i] = make_double2(1.0, 0.0);
}

inline unsigned nblk(long long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

namespace kern {

void set_float_mode(int mode) {
  if (mode < 0 || mode > 2) TDVP_THROW(TDVP_ERR_ARG, "bad complex64 GEMM mode");
  tl_float_mode = mode;
}
int float_mode() { return tl_float_mode; }

void set_kmap(const KMap* k) { tl_kmap = k; }
const KMap* current_kmap() { return tl_kmap; }

thread_local void* tl_split_ws = nullptr;
thread_local size_t tl_split_wsb = 0;
void set_split_workspace(void* p, size_t bytes) {
  tl_split_ws = p;
  tl_split_wsb = p ? bytes : 0;
}
SplitWorkspaceScope::SplitWorkspaceScope(void* p, size_t bytes) : saved_p(tl_split_ws), saved_b(tl_split_wsb) {
  set_split_workspace(p, bytes);
}
SplitWorkspaceScope::~SplitWorkspaceScope() { set_split_workspace(saved_p, saved_b); }

template <typename T>
void gemm(hipStream_t s, int opa, int opb, int M, int N, int K, zc alpha, const void* A, long long lda,
          long long sa, const void* B, long long ldb, long long sb, zc beta, void* C, long long ldc,
          long long sc, int batch, void* ws, size_t ws_bytes) {
  if (M <= 0 || N <= 0 || batch <= 0) return;
  if (!ws) {
    ws = tl_split_ws;
    ws_bytes = tl_split_wsb;
  }
  switch (opa) {
    case TDVP_OP_N: dispatch_b<T, TDVP_OP_N>(s, opb, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, ws_bytes); break;
    case TDVP_OP_T: dispatch_b<T, TDVP_OP_T>(s, opb, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, ws_bytes); break;
    case TDVP_OP_C: dispatch_b<T, TDVP_OP_C>(s, opb, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, ws_bytes); break;
    case TDVP_OP_R: dispatch_b<T, TDVP_OP_R>(s, opb, M, N, K, alpha, A, lda, sa, B, ldb, sb, beta, C, ldc, sc, batch, ws, ws_bytes); break;
    default: TDVP_THROW(TDVP_ERR_ARG, "bad GEMM op_a");
  }
  HIP_CHECK(hipGetLastError());
}
template void gemm<double>(hipStream_t, int, int, int, int, int, zc, const void*, long long, long long,
                           const void*, long long, long long, zc, void*, long long, long long, int, void*, size_t);

template <typename T>
void gemm_heff(hipStream_t s, int M, int N, int K, const void* A, long long lda, const void* B, long long ldb,
               void* C, long long ldc, void* ws, size_t ws_bytes) {
  if (M <= 0 || N <= 0) return;
  launch_gemm<T, TDVP_OP_N, TDVP_OP_N, 1>(s, M, N, K, 1.0, A, lda, 0, B, ldb, 0, 0.0, C, ldc, 0, 1, ws, ws_bytes);
  HIP_CHECK(hipGetLastError());
}
template void gemm_heff<double>(hipStream_t, int, int, int, const void*, long long, const void*, long long, void*,
                                long long, void*, size_t);
template void gemm_heff<float>(hipStream_t, int, int, int, const void*, long long, const void*, long long, void*,
                               long long, void*, size_t);

template <typename T>
void gemm_heff_batched(hipStream_t s, int M, int N, int K, const void* A, long long lda, long long sa, const void* B,
                       long long ldb, long long sb, void* C, long long ldc, long long sc, int batch) {
  if (M <= 0 || N <= 0 || batch <= 0) return;
  launch_gemm<T, TDVP_OP_N, TDVP_OP_N, 1>(s, M, N, K, 1.0, A, lda, sa, B, ldb, sb, 0.0, C, ldc, sc, batch);
  HIP_CHECK(hipGetLastError());
}
template void gemm_heff_batched<double>(hipStream_t, int, int, int, const void*, long long, long long, const void*,
                                        long long, long long, void*, long long, long long, int);
template void gemm_heff_batched<float>(hipStream_t, int, int, int, const void*, long long, long long, const void*,
                                       long long, long long, void*, long long, long long, int);

template <typename T>
void gemm_nn_ws(hipStream_t s, int M, int N, int K, zc alpha, const void* A, long long lda, const void* B,
                long long ldb, zc beta, void* C, long long ldc, void* ws, size_t ws_bytes) {
  if (M <= 0 || N <= 0) return;
  launch_gemm<T, TDVP_OP_N, TDVP_OP_N, 0>(s, M, N, K, alpha, A, lda, 0, B, ldb, 0, beta, C, ldc, 0, 1, ws,
                                          ws_bytes);
  HIP_CHECK(hipGetLastError());
}
template void gemm_nn_ws<double>(hipStream_t, int, int, int, zc, const void*, long long, const void*, long long, zc,
                                 void*, long long, void*, size_t);
template void gemm_nn_ws<float>(hipStream_t, int, int, int, zc, const void*, long long, const void*, long long, zc,
                                void*, long long, void*, size_t);
template void gemm<float>(hipStream_t, int, int, int, int, int, zc, const void*, long long, long long,
                          const void*, long long, long long, zc, void*, long long, long long, int, void*, size_t);

// Whether the stage goes through LDS, from the nonzeros an output channel has on
// average and the blocks of 64 columns of a row.  Matvecs with 32 x 32 channels,
// FP64, direct / LDS in us: chi = 512 (4096 blocks) with 4 nonzeros 2022 / 2012, 8
// 2131 / 2056, 32 2908 / 2517, 48 3229 / 2791, all 64 2786 / 3049 (every wave reads
// every input, in the same order); chi = 256 (1024 blocks) with 8 310 / 307, 32
// 433 / 433, 48 485 / 504; chi = 64 with 8 47 / 64, 32 62 / 139.  FP32: 512 with 8
// 802 / 765, 32 1189 / 1005, 64 1174 / 1284.
static bool wapply_by_lds(const WTable& t, size_t lds, long long blocks) {
  return lds <= 64 * 1024 && blocks >= 4096 && t.nnz > 6LL * t.n_out_ch && t.nnz <= 56LL * t.n_out_ch;
}
template <typename T>
void wapply(hipStream_t s, const WTable& t, const void* in, void* out, long long nP, long long nQ,
            long long isP, long long isQ, long long is1, long long is2, long long osP, long long osQ,
            long long os1, long long os2, const WCharges* wc) {
  if (nP <= 0 || nQ <= 0) return;
  if (nP > 65535) TDVP_THROW(TDVP_ERR_ARG, "wapply: P extent too large");
  if (isQ != 1 || osQ != 1) TDVP_THROW(TDVP_ERR_ARG, "wapply: columns must be contiguous");
  WCharges w{nullptr, nullptr, nullptr, nullptr, 0};
  if (wc) {
    if (!wc->ql || !wc->qr || !wc->din || !wc->dout) TDVP_THROW(TDVP_ERR_ARG, "wapply: incomplete charge table");
    w = *wc;
  }
  const WPointers dev{t.rowptr, t.col, t.val};
  auto route = [&](auto&& go) {
    if (t.inl && wc) go(std::true_type{}, *t.inl);
    else if (t.inl) go(std::false_type{}, *t.inl);
    else if (wc) go(std::true_type{}, dev);
    else go(std::false_type{}, dev);
    HIP_CHECK(hipGetLastError());
  };
  const size_t lds = (size_t)t.n_in_ch * 64 * sizeof(typename VT<T>::c2);
  if (wapply_by_lds(t, lds, (nQ + 63) / 64 * nP)) {
    const dim3 grid((unsigned)((nQ + 63) / 64), (unsigned)nP);
    return route([&](auto charged, const auto& tab) {
      hipLaunchKernelGGL((wapply_lds_kernel<T, decltype(charged)::value, std::decay_t<decltype(tab)>>), grid, dim3(WNT),
                         lds, s, static_cast<const T*>(in), static_cast<T*>(out), nQ, isP, is1, is2, osP, os1, os2, tab,
                         t.n_in_ch, t.n_out_ch, w);
    });
  }
  // about 2048 blocks of four waves fill the device; fewer rows and columns:
  // the output channels are dealt over the grid as well
  constexpr int V = sizeof(T) == 8 ? 1 : 2, WAVES = WNT / 64;
  const long long gx = (nQ + 64 * V - 1) / (64 * V);
  const long long gz = std::max<long long>(
      1, std::min<long long>((2048 + gx * nP - 1) / (gx * nP), (t.n_out_ch + WAVES - 1) / WAVES));
  const dim3 grid((unsigned)gx, (unsigned)nP, (unsigned)gz);
  route([&](auto charged, const auto& tab) {
    hipLaunchKernelGGL((wapply_kernel<T, V, decltype(charged)::value, std::decay_t<decltype(tab)>>), grid, dim3(WNT), 0,
                       s, static_cast<const T*>(in), static_cast<T*>(out), nQ, isP, is1, is2, osP, os1, os2, tab,
                       t.n_out_ch, w);
  });
}
template void wapply<double>(hipStream_t, const WTable&, const void*, void*, long long, long long, long long,
                             long long, long long, long long, long long, long long, long long, long long,
                             const WCharges*);
template void wapply<float>(hipStream_t, const WTable&, const void*, void*, long long, long long, long long,
                            long long, long long, long long, long long, long long, long long, long long,
                            const WCharges*);

int zdots_blocks(long long n) { return (int)std::max<long long>(1, (n + DOT_CHUNK - 1) / DOT_CHUNK); }

void zdots(hipStream_t s, const void* V, long long ldv, int nv, const void* w, long long n, void* partial,
           int nb, void* out, bool conjugate) {
  if (nv <= 0) return;
  if (conjugate)
    hipLaunchKernelGGL(zdots_partial_kernel<true>, dim3(nb, nv), dim3(VNT), 0, s, static_cast<const double2*>(V), ldv,
                       nv, static_cast<const double2*>(w), n, static_cast<double2*>(partial));
  else
    hipLaunchKernelGGL(zdots_partial_kernel<false>, dim3(nb, nv), dim3(VNT), 0, s, static_cast<const double2*>(V), ldv,
                       nv, static_cast<const double2*>(w), n, static_cast<double2*>(partial));
  hipLaunchKernelGGL(zdots_final_kernel, dim3(nv), dim3(VNT), 0, s,
                     static_cast<const double2*>(partial), nb, nv, static_cast<double2*>(out));
  HIP_CHECK(hipGetLastError());
}

void zsum_partials(hipStream_t s, const void* partial, int nb, int nv, void* out) {
  if (nv <= 0) return;
  hipLaunchKernelGGL(zdots_final_kernel, dim3(nv), dim3(VNT), 0, s, static_cast<const double2*>(partial), nb, nv,
                     static_cast<double2*>(out));
  HIP_CHECK(hipGetLastError());
}

int zcombine_norm_blocks(long long n) { return (int)std::max<long long>(1, nblk(n, VNT)); }

void zdots_partial(hipStream_t s, const void* V, long long ldv, int nv, const void* w, long long n, void* partial,
                   int nb) {
  if (nv <= 0) return;
  hipLaunchKernelGGL(zdots_partial_kernel<true>, dim3(nb, nv), dim3(VNT), 0, s, static_cast<const double2*>(V), ldv,
                     nv, static_cast<const double2*>(w), n, static_cast<double2*>(partial));
  HIP_CHECK(hipGetLastError());
}

void zcombine_p(hipStream_t s, void* w, const void* V, long long ldv, int nv, const void* partial, int nb,
                double sign, long long n, void* cout, void* npart) {
  if (n <= 0 || nv <= 0) return;
  if (nv > ZC_MAXV) TDVP_THROW(TDVP_ERR_ARG, "zcombine_p: at most 64 vectors");
  if (npart)
    hipLaunchKernelGGL(zcombine_p_kernel<true>, dim3(nblk(n, VNT)), dim3(VNT), 0, s, static_cast<double2*>(w),
                       static_cast<const double2*>(V), ldv, nv, static_cast<const double2*>(partial), nb, sign, n,
                       static_cast<double2*>(cout), static_cast<double2*>(npart));
  else
    hipLaunchKernelGGL(zcombine_p_kernel<false>, dim3(nblk(n, VNT)), dim3(VNT), 0, s, static_cast<double2*>(w),
                       static_cast<const double2*>(V), ldv, nv, static_cast<const double2*>(partial), nb, sign, n,
                       static_cast<double2*>(cout), nullptr);
  HIP_CHECK(hipGetLastError());
}

void zcombine_dots(hipStream_t s, void* w, const void* V, long long ldv, int nv, const void* partial, int nb,
                   double sign, long long n, void* cout, void* dpart) {
  if (n <= 0 || nv <= 0) return;
  if (nv > ZC_MAXV) TDVP_THROW(TDVP_ERR_ARG, "zcombine_dots: at most 64 vectors");
  hipLaunchKernelGGL(zcombine_dots_kernel, dim3(nblk(n, VNT)), dim3(VNT), 0, s, static_cast<double2*>(w),
                     static_cast<const double2*>(V), ldv, nv, static_cast<const double2*>(partial), nb, sign, n,
                     static_cast<double2*>(cout), static_cast<double2*>(dpart));
  HIP_CHECK(hipGetLastError());
}

void zcombine_host(hipStream_t s, void* dst, const void* V, long long ldv, int nv, const zc* c, long long n) {
  if (n <= 0) return;
  if (nv > ZC_ARGS) TDVP_THROW(TDVP_ERR_ARG, "zcombine_host: at most 64 vectors");
  CombineArgs a{};
  for (int j = 0; j < nv; ++j) a.c[j] = make_double2(c[j].real(), c[j].imag());
  hipLaunchKernelGGL(zcombine_args_kernel, dim3(nblk(n, VNT)), dim3(VNT), 0, s, static_cast<double2*>(dst),
                     static_cast<const double2*>(V), ldv, nv, a, n);
  HIP_CHECK(hipGetLastError());
}

void zscale(hipStream_t s, void* dst, const void* src, zc a, long long n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(zscale_kernel, dim3(nblk(n)), dim3(256), 0, s, static_cast<double2*>(dst),
                     static_cast<const double2*>(src), a.real(), a.imag(), n);
  HIP_CHECK(hipGetLastError());
}

void zscale_invnorm(hipStream_t s, void* w, const void* partial, int np, void* out, long long n, void* host,
                    const void* coeffs, int ncoef, int host_norm_at) {
  if (n <= 0) return;
  hipLaunchKernelGGL(zscale_invnorm_kernel, dim3(nblk(n, VNT)), dim3(VNT), 0, s, static_cast<double2*>(w),
                     static_cast<const double2*>(partial), np, static_cast<double2*>(out), n,
                     static_cast<double2*>(host), static_cast<const double2*>(coeffs), ncoef, host_norm_at);
  HIP_CHECK(hipGetLastError());
}

void z2c(hipStream_t s, void* dst, const void* src, long long n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(z2c_kernel, dim3(nblk(n)), dim3(256), 0, s, static_cast<float2*>(dst),
                     static_cast<const double2*>(src), n);
  HIP_CHECK(hipGetLastError());
}

void c2z(hipStream_t s, void* dst, const void* src, long long n) {
  if (n <= 0) return;
  hipLaunchKernelGGL(c2z_kernel, dim3(nblk(n)), dim3(256), 0, s, static_cast<double2*>(dst),
                     static_cast<const float2*>(src), n);
  HIP_CHECK(hipGetLastError());
}

void copy2d(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, long long rows,
            long long cols, int esize) {
  if (rows <= 0 || cols <= 0) return;
  if (esize == 16)
    hipLaunchKernelGGL(copy2d_kernel<double2>, dim3(nblk(rows * cols)), dim3(256), 0, s, static_cast<double2*>(dst),
                       ldd, static_cast<const double2*>(src), lds, rows, cols);
  else
    hipLaunchKernelGGL(copy2d_kernel<float2>, dim3(nblk(rows * cols)), dim3(256), 0, s, static_cast<float2*>(dst),
                       ldd, static_cast<const float2*>(src), lds, rows, cols);
  HIP_CHECK(hipGetLastError());
}

void ztri(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, long long rows,
          long long cols, int mode) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(ztri_kernel, dim3(nblk(rows * cols)), dim3(256), 0, s, static_cast<double2*>(dst), ldd,
                     static_cast<const double2*>(src), lds, rows, cols, mode);
  HIP_CHECK(hipGetLastError());
}

void zconjtrans(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, long long rows,
                long long cols) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(zconjtrans_kernel, dim3(nblk(rows * cols)), dim3(256), 0, s, static_cast<double2*>(dst),
                     ldd, static_cast<const double2*>(src), lds, rows, cols);
  HIP_CHECK(hipGetLastError());
}

void zhermitize(hipStream_t s, void* A, long long n) { zhermitize_to(s, A, A, n); }

void zhermitize_to(hipStream_t s, void* A, const void* S, long long n, int* zero, int nzero) {
  if (n <= 0) return;
  hipLaunchKernelGGL(zhermitize_kernel, dim3(nblk(n * n)), dim3(256), 0, s, static_cast<double2*>(A),
                     static_cast<const double2*>(S), n, zero, nzero);
  HIP_CHECK(hipGetLastError());
}

void zfill(hipStream_t s, void* dst, zc v, long long n, int esize) {
  if (n <= 0) return;
  if (esize == 16)
    hipLaunchKernelGGL(fill_kernel<double2>, dim3(nblk(n)), dim3(256), 0, s, static_cast<double2*>(dst),
                       make_double2(v.real(), v.imag()), n);
  else
    hipLaunchKernelGGL(fill_kernel<float2>, dim3(nblk(n)), dim3(256), 0, s, static_cast<float2*>(dst),
                       make_float2(float(v.real()), float(v.imag())), n);
  HIP_CHECK(hipGetLastError());
}

template <bool PACK>
void rows_pack_dispatch(hipStream_t s, void* packed, int pe, void* dense, int de, int rows, long long ld, const int* seg,
                        int maxlen) {
  if (rows <= 0 || maxlen <= 0) return;
  if (rows > 65535) TDVP_THROW(TDVP_ERR_ARG, "row segments: too many rows");
  const dim3 grid((unsigned)((maxlen + 255) / 256), (unsigned)rows);
  if (pe == 16 && de == 16)
    hipLaunchKernelGGL((rows_pack_kernel<double2, double2, PACK>), grid, dim3(256), 0, s, static_cast<double2*>(packed),
                       static_cast<double2*>(dense), rows, ld, seg);
  else if (pe == 16 && de == 8)
    hipLaunchKernelGGL((rows_pack_kernel<double2, float2, PACK>), grid, dim3(256), 0, s, static_cast<double2*>(packed),
                       static_cast<float2*>(dense), rows, ld, seg);
  else
    TDVP_THROW(TDVP_ERR_ARG, "row segments: unsupported element sizes");
  HIP_CHECK(hipGetLastError());
}
void pack_rows(hipStream_t s, void* packed, int packed_esize, const void* dense, int dense_esize, int rows, long long ld,
               const int* seg, int maxlen) {
  rows_pack_dispatch<true>(s, packed, packed_esize, const_cast<void*>(dense), dense_esize, rows, ld, seg, maxlen);
}
void unpack_rows(hipStream_t s, void* dense, int dense_esize, const void* packed, int packed_esize, int rows,
                 long long ld, const int* seg, int maxlen) {
  rows_pack_dispatch<false>(s, const_cast<void*>(packed), packed_esize, dense, dense_esize, rows, ld, seg, maxlen);
}

void zrandom_blocks(hipStream_t s, void* E, int R, int C, const int* qr, const int* qc, unsigned long long seed) {
  const long long n = (long long)R * C;
  if (n <= 0) return;
  hipLaunchKernelGGL(zrandom_blocks_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, static_cast<double2*>(E),
                     R, C, qr, qc, seed);
  HIP_CHECK(hipGetLastError());
}

void zscale_phys(hipStream_t s, void* G, long long nx, long long nq, double f0, double f1) {
  if (nx <= 0 || nq <= 0) return;
  hipLaunchKernelGGL(zscale_phys_kernel, dim3(nblk(nx * 2 * nq)), dim3(256), 0, s, static_cast<double2*>(G),
                     nx, nq, f0, f1);
  HIP_CHECK(hipGetLastError());
}

void zshift_diag(hipStream_t s, void* G, long long n, double a, double b) {
  if (n <= 0) return;
  hipLaunchKernelGGL(zshift_diag_kernel, dim3(nblk(n * n)), dim3(256), 0, s, static_cast<double2*>(G), n, a, b);
  HIP_CHECK(hipGetLastError());
}

void zscale_rows(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, long long rows,
                 long long cols, const double* f) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(zscale_rc_kernel, dim3(nblk(rows * cols)), dim3(256), 0, s, static_cast<double2*>(dst), ldd,
                     static_cast<const double2*>(src), lds, rows, cols, f, 0);
  HIP_CHECK(hipGetLastError());
}

void zscale_cols(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, long long rows,
                 long long cols, const double* f) {
  if (rows <= 0 || cols <= 0) return;
  hipLaunchKernelGGL(zscale_rc_kernel, dim3(nblk(rows * cols)), dim3(256), 0, s, static_cast<double2*>(dst), ldd,
                     static_cast<const double2*>(src), lds, rows, cols, f, 1);
  HIP_CHECK(hipGetLastError());
}

void zgather(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, const int* ridx, long long nr,
             const int* cidx, long long nc) {
  if (nr <= 0 || nc <= 0) return;
  hipLaunchKernelGGL(zgather_kernel, dim3(nblk(nr * nc)), dim3(256), 0, s, static_cast<double2*>(dst), ldd,
                     static_cast<const double2*>(src), lds, ridx, nr, cidx, nc);
  HIP_CHECK(hipGetLastError());
}

void zscatter(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, const int* ridx, long long nr,
              const int* cidx, long long nc) {
  if (nr <= 0 || nc <= 0) return;
  hipLaunchKernelGGL(zscatter_kernel, dim3(nblk(nr * nc)), dim3(256), 0, s, static_cast<double2*>(dst), ldd,
                     static_cast<const double2*>(src), lds, ridx, nr, cidx, nc);
  HIP_CHECK(hipGetLastError());
}

void zscatter_cols(hipStream_t s, void* dst, long long ldd, const void* src, long long lds, long long nr,
                   const int* cidx, long long nc) {
  zscatter(s, dst, ldd, src, lds, nullptr, nr, cidx, nc);
}

void zunit_blocks(hipStream_t s, void* diag, const void* H, long long n, const int* idx, const int* pos, int cnt,
                  void* rows) {
  if (cnt <= 0) return;
  hipLaunchKernelGGL(zunit_blocks_kernel, dim3(nblk(cnt)), dim3(256), 0, s, static_cast<double2*>(diag),
                     static_cast<const double2*>(H), n, idx, pos, cnt, static_cast<double2*>(rows));
  HIP_CHECK(hipGetLastError());
}

}  // namespace kern
