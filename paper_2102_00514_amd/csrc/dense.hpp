// Wavefront-cooperative form of the method for larger states (n = 20): one
// 64-lane workgroup owns one element at a time, with its N x N matrices in
// LDS, and the scans run as a hierarchy of chunk folds (Section 4, eq. 15 and
// eq. 19 evaluated as in operators.hpp; elements as in elements.hpp).
//
// HBM records are slot-major (all words of one slot contiguous), so a wave
// reads or writes one record with contiguous lanes.  Symmetric matrices are
// stored upper-packed (sym_index order) in HBM and full in LDS.
#pragma once

#include <type_traits>

#include "elements.hpp"
#include "slot_kernels.hpp"

namespace pks {
namespace dn {

constexpr int kWave = 64;

template <int N>
constexpr int ld() { return N + 1; }           // LDS row length (odd: spreads banks)
template <int N>
constexpr int mat_words() { return N * ld<N>(); }

// The lane, opaque to the optimiser at every call: a routine computes its LDS
// addresses when it runs.  Left visible, the addresses of every routine of a
// kernel are hoisted out of its slot loop and spill to scratch around each
// factorisation: k_dn_forward_down_backward_up 1.63 ms (416 bytes of scratch
// per lane) against 1.24 and k_dn_forward_up 1.57 against 1.13 at 65,537 slots.
// The smoothing kernels, which factorise nothing, are 12 % slower by it.
PKS_DEV int lane() {
  int l = int(threadIdx.x);
  asm volatile("" : "+v"(l));
  return l;
}
PKS_DEV void wsync() { __syncthreads(); }     // workgroups are a single wave

// ---------------------------------------------------------------------------
// Wave-wide matrix routines on LDS operands (leading dimension ld<LDN>()).
// Each ends with a barrier, so its results are visible to every lane.
// ---------------------------------------------------------------------------

typedef double f64x4 __attribute__((ext_vector_type(4)));

// The VALU form of mm below: each lane computes a 2 x 4 block of C, so every
// LDS word it loads feeds two or four multiply-adds.
template <int LDN, int M, int K, int NC, bool TA, bool TB, typename R>
PKS_DEV void mm_valu(const R* A, const R* B, const R* C0, R sgn, R* C) {
  constexpr int L = ld<LDN>();
  constexpr int TR = 2, TC = 4;
  constexpr int MR = (M + TR - 1) / TR, MC = (NC + TC - 1) / TC;
  for (int t = lane(); t < MR * MC; t += kWave) {
    const int i0 = (t / MC) * TR, j0 = (t % MC) * TC;
    R acc[TR][TC];
    PKS_UNROLL for (int r = 0; r < TR; ++r) PKS_UNROLL for (int c = 0; c < TC; ++c) acc[r][c] = R(0);
#pragma unroll 4
    for (int k = 0; k < K; ++k) {
      R a[TR], b[TC];
      PKS_UNROLL for (int r = 0; r < TR; ++r) {
        const int i = i0 + r;
        a[r] = (M % TR == 0 || i < M) ? (TA ? A[k * L + i] : A[i * L + k]) : R(0);
      }
      PKS_UNROLL for (int c = 0; c < TC; ++c) {
        const int j = j0 + c;
        b[c] = (NC % TC == 0 || j < NC) ? (TB ? B[j * L + k] : B[k * L + j]) : R(0);
      }
      PKS_UNROLL for (int r = 0; r < TR; ++r) PKS_UNROLL for (int c = 0; c < TC; ++c)
        acc[r][c] = fma(a[r], b[c], acc[r][c]);
    }
    PKS_UNROLL for (int r = 0; r < TR; ++r) PKS_UNROLL for (int c = 0; c < TC; ++c) {
      const int i = i0 + r, j = j0 + c;
      if ((M % TR == 0 || i < M) && (NC % TC == 0 || j < NC))
        C[i * L + j] = (C0 ? C0[i * L + j] : R(0)) + sgn * acc[r][c];
    }
  }
  wsync();
}

// y = y0 + sgn * op(A) x, op(A) M x K.  y may alias y0 but not x.
template <int LDN, int M, int K, bool TA, typename R, bool SYNC = true>
PKS_DEV void mv(const R* A, const R* x, const R* y0, R sgn, R* y) {
  constexpr int L = ld<LDN>();
  for (int i = lane(); i < M; i += kWave) {
    R s = R(0);
    PKS_UNROLL for (int k = 0; k < K; ++k) s = fma(TA ? A[k * L + i] : A[i * L + k], x[k], s);
    y[i] = (y0 ? y0[i] : R(0)) + sgn * s;
  }
  if constexpr (SYNC) wsync();
}

// C = C0 + sgn * op(A) op(B), op(A) M x K, op(B) K x NC.  C may alias C0 but
// not A or B.  C0 may be null (zero).  FP64: on the matrix cores; FP32:
// mm_valu.
//
// 20 x K x 20 (the full-state blocks): 16 x 16 of the result with
// v_mfma_f64_16x16x4f64 and its last four rows and columns with
// v_mfma_f64_4x4x4f64, whose four independent 4 x 4 blocks are the row (or
// column) tiles of the strip.  Lane l feeds A[l % 16][l / 16] and B[l / 16][l %
// 16] to both, so the strips use the operand registers of the 16 x 16 block
// and one more row and column of four; it receives D[4 q + l / 16][l % 16], q =
// 0..3, of the large form and, of block b = l / 4 % 4 of the small one,
// D_b[l / 16][l % 4].  Four large and twelve small instructions per 16 of the
// reduction take 560 cycles of the matrix core for K = 20; padding the product
// to 32 x 32 (20 large ones) took 1280, and stored and read back 2.3 times the
// result words.  One product alone on a wave: 1992 cycles before, 1080 now.
// Other shapes (multiples of four): small form alone, four result tiles per
// instruction.
//
// x, y: y = y0 + ysgn * op(A) x beside the product (x null: none), y0 may be
// null or y, but not x.  On the matrix cores the vector is one more column
// tile (every column of it the vector), which shares the product's operand
// reads and latency; alone (mv) it took 520 cycles of one wave.
template <int LDN, int M, int K, int NC, bool TA, bool TB, typename R>
PKS_DEV void mm(const R* A, const R* B, const R* C0, R sgn, R* C, const R* x = nullptr, const R* y0 = nullptr,
                R ysgn = R(1), R* y = nullptr) {
  constexpr int L = ld<LDN>();
  if constexpr (sizeof(R) == 8 && M % 4 == 0 && K % 4 == 0 && NC % 4 == 0) {
    constexpr int KS = K / 4;
    const int ln = lane(), kq = ln >> 4, c4 = ln & 3;
    auto ra = [&](int i, int k) { return double(TA ? A[k * L + i] : A[i * L + k]); };
    auto rb = [&](int k, int j) { return double(TB ? B[j * L + k] : B[k * L + j]); };
    if constexpr (M == 20 && NC == 20) {
      // every LDS read is issued before the first MFMA
      const int r = ln & 15, b4 = (ln >> 2) & 3;
      double a16[KS], a4[KS], b16[KS], bs[KS];
      PKS_UNROLL for (int ks = 0; ks < KS; ++ks) {
        const int k = 4 * ks + kq;
        a16[ks] = ra(r, k);
        b16[ks] = rb(k, r);
        a4[ks] = ra(16 + c4, k);
        bs[ks] = rb(k, 16 + c4);
      }
      int at[7];
      R c0[7];
      PKS_UNROLL for (int q = 0; q < 4; ++q) at[q] = (4 * q + kq) * L + r;
      at[4] = (4 * b4 + kq) * L + 16 + c4;   // rows 0..15, columns 16..19
      at[5] = (16 + kq) * L + r;             // rows 16..19, columns 0..15
      at[6] = (16 + kq) * L + 16 + c4;       // the corner, in every block alike
      PKS_UNROLL for (int q = 0; q < 7; ++q) c0[q] = C0 ? C0[at[q]] : R(0);
      double xs[KS], z0 = 0.0, z1 = 0.0, ya = 0.0, yb = 0.0;
      if (x) {
        PKS_UNROLL for (int ks = 0; ks < KS; ++ks) xs[ks] = x[4 * ks + kq];
        if (y0) {
          z0 = y0[4 * b4 + kq];
          z1 = y0[16 + kq];
        }
      }
      f64x4 acc = f64x4{0.0, 0.0, 0.0, 0.0};
      double right = 0.0, below = 0.0, corner = 0.0;
      PKS_UNROLL for (int ks = 0; ks < KS; ++ks) {
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a16[ks], b16[ks], acc, 0, 0, 0);
        right = __builtin_amdgcn_mfma_f64_4x4x4f64(a16[ks], bs[ks], right, 0, 0, 0);
        below = __builtin_amdgcn_mfma_f64_4x4x4f64(a4[ks], b16[ks], below, 0, 0, 0);
        corner = __builtin_amdgcn_mfma_f64_4x4x4f64(a4[ks], bs[ks], corner, 0, 0, 0);
        if (x) {
          ya = __builtin_amdgcn_mfma_f64_4x4x4f64(a16[ks], xs[ks], ya, 0, 0, 0);
          yb = __builtin_amdgcn_mfma_f64_4x4x4f64(a4[ks], xs[ks], yb, 0, 0, 0);
        }
      }
      PKS_UNROLL for (int q = 0; q < 4; ++q) C[at[q]] = c0[q] + sgn * R(acc[q]);
      C[at[4]] = c0[4] + sgn * R(right);
      C[at[5]] = c0[5] + sgn * R(below);
      C[at[6]] = c0[6] + sgn * R(corner);
      if (x) {
        y[4 * b4 + kq] = z0 + ysgn * ya;
        y[16 + kq] = z1 + ysgn * yb;
      }
    } else {
      constexpr int TN = NC / 4, tiles = (M / 4) * TN, G = (tiles + 3) / 4;
      double acc[G], av[G][KS], bv[G][KS];
      int at[G];
      R c0[G];
      PKS_UNROLL for (int g = 0; g < G; ++g) {
        // blocks past the last tile compute it once more
        const int t = 4 * g + ((ln >> 2) & 3), id = t < tiles ? t : tiles - 1;
        const int i0 = 4 * (id / TN), j0 = 4 * (id % TN);
        PKS_UNROLL for (int ks = 0; ks < KS; ++ks) {
          av[g][ks] = ra(i0 + c4, 4 * ks + kq);
          bv[g][ks] = rb(4 * ks + kq, j0 + c4);
        }
        at[g] = (i0 + kq) * L + j0 + c4;
        c0[g] = C0 ? C0[at[g]] : R(0);
        acc[g] = 0.0;
      }
      static_assert(M <= 16, "row tiles of the vector fit the four blocks");
      const int iv = 4 * min((ln >> 2) & 3, M / 4 - 1);
      double ax[KS], xs[KS], z0 = 0.0, ya = 0.0;
      if (x) {
        PKS_UNROLL for (int ks = 0; ks < KS; ++ks) {
          ax[ks] = ra(iv + c4, 4 * ks + kq);
          xs[ks] = x[4 * ks + kq];
        }
        if (y0) z0 = y0[iv + kq];
      }
      PKS_UNROLL for (int ks = 0; ks < KS; ++ks) {
        PKS_UNROLL for (int g = 0; g < G; ++g)
          acc[g] = __builtin_amdgcn_mfma_f64_4x4x4f64(av[g][ks], bv[g][ks], acc[g], 0, 0, 0);
        if (x) ya = __builtin_amdgcn_mfma_f64_4x4x4f64(ax[ks], xs[ks], ya, 0, 0, 0);
      }
      PKS_UNROLL for (int g = 0; g < G; ++g) C[at[g]] = c0[g] + sgn * R(acc[g]);
      if (x) y[iv + kq] = z0 + ysgn * ya;
    }
    wsync();
    return;
  }
  if (x) mv<LDN, M, K, TA, R, false>(A, x, y0, ysgn, y);
  mm_valu<LDN, M, K, NC, TA, TB, R>(A, B, C0, sgn, C);
}

// Value of x in lane `src` (uniform), as a double.
PKS_DEV double lane_value(double x, int src) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane(int(v & 0xffffffffll), src);
  const int hi = __builtin_amdgcn_readlane(int(v >> 32), src);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// Left-looking factorisation with the library square root and division, a
// column at a time in LDS: chol for pivots outside the range of its fast form
// (not positive, not finite, or so large or small that its residuals would
// leave the exponent range).
template <int LDN, int N, typename R>
PKS_DEV void chol_any(R* A, int* ok) {
  constexpr int L = ld<LDN>();
  const int i = lane();
  bool good = true;
#pragma unroll 1
  for (int j = 0; j < N; ++j) {
    R s = R(0);
    if (i < N) {
      s = A[i * L + j];
#pragma unroll 1
      for (int t = 0; t < j; ++t) s = fma(-A[i * L + t], A[j * L + t], s);
    }
    const R d = R(lane_value(double(s), j));
    good = good && d > R(0);
    const R sd = sqrt(d);
    wsync();                                     // row j has been read
    if (i < N) A[i * L + j] = i == j ? sd : (i > j ? s / sd : R(0));
    wsync();
  }
  if (i == 0 && !good) *ok = 0;
}

// f(std::integral_constant<int, B>) ... f(<E - 1>): loops whose index selects a
// cross-lane move, which takes it as an instruction field.
template <int B, int E, class F>
PKS_DEV void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// The value of lane SRC of each row of 16 lanes, in every lane of that row
// (row_newbcast, on the VALU).  Reading a lane through the scalar unit instead
// stalls its user by about 20 cycles.
template <int SRC>
PKS_DEV double row_bcast(double x) { return __builtin_amdgcn_mov_dpp(x, 0x150 + SRC, 0xf, 0xf, true); }
template <int SRC>
PKS_DEV float row_bcast(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x150 + SRC, 0xf, 0xf, true));
}

// A lower-triangular N x N factor in registers, N even, N / 2 <= 16: lane l
// holds rows l % 16 and l % 16 + N / 2 (the first without its columns past N /
// 2), every 16 lanes the same, so that an entry reaches all lanes by one
// row_bcast; lanes l % 16 >= N / 2 repeat row N / 2 - 1 and the last.  The
// diagonal entries of the two rows stand in dlo and dhi (those of lo and hi are
// not used), their reciprocals in rlo and rhi.
template <int N, typename R>
struct Factor {
  static constexpr int H = N / 2;
  static_assert(N % 2 == 0 && H <= 16, "two rows per lane of a row of 16");
  R lo[H], hi[N], dlo, dhi;
  double rlo, rhi;
  static PKS_DEV int row(int l) { return min(l & 15, H - 1); }
  // entry (K, K) and its reciprocal, in every lane
  template <int K>
  PKS_DEV R diag() const { return K < H ? row_bcast<K % H>(dlo) : row_bcast<K % H>(dhi); }
  template <int K>
  PKS_DEV double rcp() const { return K < H ? row_bcast<K % H>(rlo) : row_bcast<K % H>(rhi); }
  template <int LDN>
  PKS_DEV void load(const R* A) {
    constexpr int L = ld<LDN>();
    const int rl = row(lane());
    const R *a = A + rl * L, *b = a + H * L;
    PKS_UNROLL for (int k = 0; k < H; ++k) lo[k] = a[k];
    PKS_UNROLL for (int k = 0; k < N; ++k) hi[k] = b[k];
    dlo = a[rl];
    dhi = b[rl + H];
    rlo = 1.0 / double(dlo);
    rhi = 1.0 / double(dhi);
  }
};

// Multiply-adds whose first factor comes over from another lane of the row of
// 16 (one instruction each, 5 cycles).  fnma_lanes: acc[u] -= (src of lane LANE
// + u) * x, u < CNT <= 10; fnma_sum: acc -= sum over u, in order, of (src of
// lane LANE + u) * x[u].  The two wait states that a lane move needs after its
// source was written stand at the head of the block, and nothing in the block
// writes src.
#define PKS_T(T, d, x, u) "v_fmac_" T "_dpp %" d ", -%[s], %" x " row_newbcast:%[l]+" #u " row_mask:0xf bank_mask:0xf\n\t"
#define PKS_V1(F, T) F(T, 0)
#define PKS_V2(F, T) PKS_V1(F, T) F(T, 1)
#define PKS_V3(F, T) PKS_V2(F, T) F(T, 2)
#define PKS_V4(F, T) PKS_V3(F, T) F(T, 3)
#define PKS_V5(F, T) PKS_V4(F, T) F(T, 4)
#define PKS_V6(F, T) PKS_V5(F, T) F(T, 5)
#define PKS_V7(F, T) PKS_V6(F, T) F(T, 6)
#define PKS_V8(F, T) PKS_V7(F, T) F(T, 7)
#define PKS_V9(F, T) PKS_V8(F, T) F(T, 8)
#define PKS_V10(F, T) PKS_V9(F, T) F(T, 9)
#define PKS_O1(c, v) [v0] c(v[0])
#define PKS_O2(c, v) PKS_O1(c, v), [v1] c(v[1])
#define PKS_O3(c, v) PKS_O2(c, v), [v2] c(v[2])
#define PKS_O4(c, v) PKS_O3(c, v), [v3] c(v[3])
#define PKS_O5(c, v) PKS_O4(c, v), [v4] c(v[4])
#define PKS_O6(c, v) PKS_O5(c, v), [v5] c(v[5])
#define PKS_O7(c, v) PKS_O6(c, v), [v6] c(v[6])
#define PKS_O8(c, v) PKS_O7(c, v), [v7] c(v[7])
#define PKS_O9(c, v) PKS_O8(c, v), [v8] c(v[8])
#define PKS_O10(c, v) PKS_O9(c, v), [v9] c(v[9])
#define PKS_FL(T, u) PKS_T(T, "[v" #u "]", "[x]", u)
#define PKS_FS(T, u) PKS_T(T, "[a]", "[v" #u "]", u)
#define PKS_LANES(T, n) \
  if constexpr (CNT == n) asm("s_nop 1\n\t" PKS_V##n(PKS_FL, T) : PKS_O##n("+v", acc) : [s] "v"(src), [x] "v"(x), [l] "n"(LANE));
#define PKS_SUM(T, n) \
  if constexpr (CNT == n) asm("s_nop 1\n\t" PKS_V##n(PKS_FS, T) : [a] "+v"(acc) : [s] "v"(src), PKS_O##n("v", x), [l] "n"(LANE));
#define PKS_ALL(F, T) \
  F(T, 1) F(T, 2) F(T, 3) F(T, 4) F(T, 5) F(T, 6) F(T, 7) F(T, 8) F(T, 9) F(T, 10)
#define PKS_FNMA(R, T)                                                           \
  template <int LANE, int CNT>                                                   \
  PKS_DEV void fnma_lanes(R* acc, R src, R x) {                                  \
    static_assert(CNT >= 1 && CNT <= 10 && LANE + CNT <= 16, "lanes of one row"); \
    PKS_ALL(PKS_LANES, T)                                                        \
  }                                                                              \
  template <int LANE, int CNT>                                                   \
  PKS_DEV void fnma_sum(R& acc, R src, const R* x) {                             \
    static_assert(CNT >= 1 && CNT <= 10 && LANE + CNT <= 16, "lanes of one row"); \
    PKS_ALL(PKS_SUM, T)                                                          \
  }
PKS_FNMA(double, "f64")
PKS_FNMA(float, "f32")
#undef PKS_FNMA

// Lower Cholesky factor (true diagonal) of the matrix A in LDS, into f and,
// with store, in place of A, the upper triangle cleared.  *ok (LDS) is cleared
// when a pivot is not positive; the factor then holds NaN, which reaches the
// convergence statistic.  Only the lower triangle of A is read.
//
// A finished column is applied to the later ones at once, to the next one
// first: the others (in blocks of fnma_lanes) fill the gaps of the chain from
// pivot to pivot (sum, broadcast, square root, quotient, product).  The sums
// of even and odd columns stay apart and are added last.  Entries above the
// diagonal hold unused values until the factor is stored.  Square root and
// quotients share one estimate y of 1/sqrt(d): the hardware's (5e-8) after one
// Newton step (4e-15); with g = d y, g + (d - g^2) y / 2 is the correctly
// rounded root, and with q = s y, q + (s - q root) y the correctly rounded
// quotient (Markstein's corrections: what y lacks enters squared), in 9
// dependent operations where the library root and division took about 30.
// One factorisation alone on a wave: 9280 cycles before, 4870 now.
template <int LDN, int N, typename R>
PKS_DEV void chol(R* A, int* ok, Factor<N, R>& f, bool store) {
  constexpr int L = ld<LDN>(), H = N / 2;
  const int ln = lane(), rl = Factor<N, R>::row(ln);
  const R *Al = A + rl * L, *Ah = Al + H * L;
  R lodd[H], hodd[N];
  PKS_UNROLL for (int k = 0; k < H; ++k) {
    f.lo[k] = Al[k];
    lodd[k] = R(0);
  }
  PKS_UNROLL for (int k = 0; k < N; ++k) {
    f.hi[k] = Ah[k];
    hodd[k] = R(0);
  }
  f.rlo = f.rhi = 0.0;
  R dl = R(0), dh = R(0);    // diagonal entries of the two rows
  // pivots of the fast form lie in [2^-664, 2^664): high words from kLow on
  constexpr unsigned kLow = 0x16700000u, kSpan = 0x69700000u - kLow;
  unsigned range = 0u;
  auto column = [&](auto J) {
    constexpr int j = decltype(J)::value, i = j > 0 ? j - 1 : 0;
    constexpr bool low = j < H;
    // column i applied to column j, and (block) to the later ones of the rows
    // that have them: part 0 the first rows, 1 the others up to column H, 2 the
    // others from H on
    if constexpr (j > 0) {
      const R l = row_bcast<j % H>(low ? f.lo[i < H ? i : 0] : f.hi[i]);
      R& ah = i & 1 ? hodd[j] : f.hi[j];
      ah = fma(-l, f.hi[i], ah);
      if constexpr (low) {
        R& al = i & 1 ? lodd[low ? j : 0] : f.lo[low ? j : 0];
        al = fma(-l, f.lo[i], al);
      }
    }
    auto block = [&](auto PT) {
      constexpr int part = decltype(PT)::value;
      constexpr int end = part < 2 ? H : N, beg = part < 2 ? 0 : H;
      constexpr int k0 = j + 1 > beg ? j + 1 : beg;
      if constexpr (j > 0 && k0 < end) {
        const R src = part < 2 ? f.lo[i < H ? i : 0] : f.hi[i];
        const R x = part == 0 ? f.lo[i < H ? i : 0] : f.hi[i];
        R* even = part == 0 ? f.lo : f.hi;
        R* odd = part == 0 ? lodd : hodd;
        fnma_lanes<k0 - beg, end - k0>((i & 1 ? odd : even) + k0, src, x);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    const R sl = low ? f.lo[low ? j : 0] + lodd[low ? j : 0] : R(0), sh = f.hi[j] + hodd[j];
    block(std::integral_constant<int, 2>{});
    const double d = double(row_bcast<j % H>(low ? sl : sh));   // pivot of column j
    double y = __builtin_amdgcn_rsq(d);
    block(std::integral_constant<int, 0>{});
    y = fma(0.5 * y, fma(-d * y, y, 1.0), y);
    const double g = d * y, hy = 0.5 * y;
    double qh = double(sh) * y, ql = double(sl) * y;
    block(std::integral_constant<int, 1>{});
    const R root = R(fma(fma(-g, g, d), hy, g));
    const double rt = double(root);
    // in FP32 the rounding of the root leaves the quotients 2^-24 off: one more correction
    if constexpr (sizeof(R) == 4) {
      qh = fma(fma(-qh, rt, double(sh)), y, qh);
      if constexpr (low) ql = fma(fma(-ql, rt, double(sl)), y, ql);
    }
    const double wh = fma(-qh, rt, double(sh)), wl = fma(-ql, rt, double(sl));
    const unsigned top = static_cast<unsigned>(static_cast<unsigned long long>(__double_as_longlong(d)) >> 32) - kLow;
    range = top > range ? top : range;
    qh = fma(wh, y, qh);
    if constexpr (low) ql = fma(wl, y, ql);
    if constexpr (low) f.lo[j] = R(ql);
    f.hi[j] = R(qh);
    const double er = fma(-rt, y, 1.0);
    const double rc = fma(sizeof(R) == 4 ? fma(er, er, er) : er, y, y);   // 1 / root
    const bool own = rl == (low ? j : j - H);
    if constexpr (low) {
      f.rlo = own ? rc : f.rlo;
      dl = own ? root : dl;
    } else {
      f.rhi = own ? rc : f.rhi;
      dh = own ? root : dh;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  static_for<0, N>(column);
  if (!__all(range < kSpan)) {     // also a pivot that is negative or not finite
    wsync();
    chol_any<LDN, N, R>(A, ok);
    f.template load<LDN>(A);
    wsync();
    return;
  }
  f.dlo = dl;
  f.dhi = dh;
  if (store) {
    // 16 lanes store the first rows, the next 16 the others
    if ((ln & 15) < H && ln < 32) {
      const bool first = ln < 16;
      const R diag = first ? dl : dh;
      R* o = A + (first ? rl : rl + H) * L;
      PKS_UNROLL for (int k = 0; k < H; ++k) o[k] = first ? (k < rl ? f.lo[k] : R(0)) : f.hi[k];
      PKS_UNROLL for (int k = H; k < N; ++k) o[k] = first || k - H >= rl ? R(0) : f.hi[k];
      o[first ? rl : rl + H] = diag;
    }
  }
  wsync();
}

template <int LDN, int N, typename R>
PKS_DEV void chol(R* A, int* ok) {
  Factor<N, R> f;
  chol<LDN, N>(A, ok, f, true);
}

// x <- Lc^-1 x and x <- Lc^-T x for one vector per lane, in registers; the
// sums run in the order of the rows they come from (ascending).  An FP64
// multiply-add issues every 4 cycles and its result is ready after 5, so the
// chains cost no more than their instructions.
template <int N>
PKS_DEV void quotient(const Factor<N, double>&, double& x, double d, double r) {
  const double q = x * r;                      // Markstein's correction: rounded as a division
  x = fma(fma(-q, d, x), r, q);
}
template <int N>
PKS_DEV void quotient(const Factor<N, float>&, float& x, float, double r) { x = float(double(x) * r); }

template <int N, typename R>
PKS_DEV void solve_l(const Factor<N, R>& f, R (&x)[N]) {
  constexpr int H = N / 2;
  static_for<0, N>([&](auto T) {
    constexpr int t = decltype(T)::value, n = t + 1;
    quotient(f, x[t], f.template diag<t>(), f.template rcp<t>());
    if constexpr (n < H) fnma_lanes<n % H, n < H ? H - n : 0>(x + n, f.lo[n < H ? t : 0], x[t]);
    constexpr int m = n > H ? n : H;   // rows of the upper half
    if constexpr (m < N) fnma_lanes<m % H, N - m>(x + m, f.hi[t], x[t]);
    __builtin_amdgcn_sched_barrier(0);
  });
}

template <int N, typename R>
PKS_DEV void solve_lt(const Factor<N, R>& f, R (&x)[N]) {
  constexpr int H = N / 2;
  static_for<0, N>([&](auto V) {
    constexpr int i = N - 1 - decltype(V)::value, n = i + 1;
    if constexpr (n < H) fnma_sum<n % H, n < H ? H - n : 0>(x[i], f.lo[n < H ? i : 0], x + n);
    constexpr int m = n > H ? n : H;
    if constexpr (m < N) fnma_sum<m % H, N - m>(x[i], f.hi[i], x + m);
    quotient(f, x[i], f.template diag<i>(), f.template rcp<i>());
    __builtin_amdgcn_sched_barrier(0);
  });
}

// A vector of N words in LDS per lane: entry i at p[i * st]; lanes without one
// read some other lane's and store nothing.
template <typename R>
struct Vec {
  R* p;
  int st;
  bool live;
  template <int N>
  PKS_DEV void get(R (&x)[N]) const { PKS_UNROLL for (int i = 0; i < N; ++i) x[i] = p[i * st]; }
  template <int N>
  PKS_DEV void put(const R (&x)[N]) const {
    if (live) {
      PKS_UNROLL for (int i = 0; i < N; ++i) p[i * st] = x[i];
    }
  }
};
// Columns 0 .. NC - 1 of B for the lanes from `first` on, as lane ln sees it.
template <int LDN, int NC, typename R>
PKS_DEV Vec<R> columns(int ln, R* B, int first = 0) {
  const int c = ln - first;
  const bool live = c >= 0 && c < NC;
  return Vec<R>{B + (live ? c : 0), ld<LDN>(), live};
}

// B <- L^-1 B, B N x NC, and x <- L^-1 x of one vector (null: none) beside it.
template <int LDN, int NC, int N, typename R>
PKS_DEV void fwd(const Factor<N, R>& f, R* B, R* x = nullptr) {
  static_assert(NC < kWave, "a lane per column, one for the vector");
  const int ln = lane();
  Vec<R> v = columns<LDN, NC>(ln, B);
  if (x && ln == NC) v = Vec<R>{x, 1, true};
  R c[N];
  v.get(c);
  solve_l(f, c);
  v.put(c);
  wsync();
}

// The same for two matrices and a vector.
template <int LDN, int NC, int N, typename R>
PKS_DEV void fwd2(const Factor<N, R>& f, R* B1, R* B2, R* x) {
  static_assert(2 * NC < kWave, "a lane per column, one for the vector");
  const int ln = lane();
  Vec<R> v = ln < NC ? columns<LDN, NC>(ln, B1) : columns<LDN, NC>(ln, B2, NC);
  if (ln == 2 * NC) v = Vec<R>{x, 1, true};
  R c[N];
  v.get(c);
  solve_l(f, c);
  v.put(c);
  wsync();
}

// B <- L^-1 U^T, U N x N.
template <int LDN, int N, typename R>
PKS_DEV void fwd_t(const Factor<N, R>& f, const R* U, R* B) {
  const int ln = lane();
  const Vec<R> v = columns<LDN, N>(ln, B);
  const R* u = U + (v.live ? ln : 0) * ld<LDN>();
  R c[N];
  PKS_UNROLL for (int i = 0; i < N; ++i) c[i] = u[i];
  solve_l(f, c);
  v.put(c);
  wsync();
}

// x <- Lc^-1 x for one vector, Lc in LDS.
template <int LDN, int N, typename R>
PKS_DEV void fwd_vec(const R* Lc, R* x) {
  Factor<N, R> f;
  f.template load<LDN>(Lc);
  const Vec<R> v{x, 1, lane() == 0};
  R c[N];
  v.get(c);
  wsync();
  solve_l(f, c);
  v.put(c);
  wsync();
}

// B <- Lc^-T B (back substitution), Lc in LDS; lane per column.
template <int LDN, int N, int NC, typename R>
PKS_DEV void bwd(const R* Lc, R* B) {
  static_assert(NC <= kWave, "a lane per column");
  Factor<N, R> f;
  f.template load<LDN>(Lc);
  const Vec<R> v = columns<LDN, NC>(lane(), B);
  R c[N];
  v.get(c);
  solve_lt(f, c);
  v.put(c);
  wsync();
}

// Lane mapping of the element-by-element routines: the lanes take whole rows
// of NC entries, kWave / NC rows per pass, so that a lane's entries are a
// constant number of rows apart (one address, immediate offsets, no division
// per entry).  f(pass, i, j) runs with row i = first row + pass * rows.
template <int M, int NC>
struct Rows {
  static constexpr int per = kWave / NC;             // rows per pass
  static constexpr int passes = (M + per - 1) / per;
  int i0, j;
  PKS_DEV Rows() {
    const int l = lane();
    i0 = l / NC;
    j = l - i0 * NC;
  }
  // whether this lane has an entry in pass r
  PKS_DEV bool live(int r) const { return i0 < per && (M % per == 0 || r + 1 < passes || i0 + r * per < M); }
};

// A <- (A + A^T) / 2
template <int LDN, int N, typename R>
PKS_DEV void symmetrize(R* A) {
  // all reads issued before the first store (one LDS latency, not one per
  // pass); both entries of a pair form the same sum
  constexpr int L = ld<LDN>();
  using Rw = Rows<N, N>;
  const Rw w;
  const int i0 = w.i0 < Rw::per ? w.i0 : 0;
  const R *a = A + i0 * L + w.j, *at = A + w.j * L + i0;
  R v[Rw::passes];
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r) {
    const int q = w.live(r) ? r : 0;
    v[r] = R(0.5) * (a[q * Rw::per * L] + at[q * Rw::per]);
  }
  R* o = A + i0 * L + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) o[r * Rw::per * L] = v[r];
  wsync();
}

template <int LDN, int M, int NC, bool TR, typename R>
PKS_DEV void copy(const R* A, R* B) {   // B = op(A), M x NC
  // all reads issued before the first store, as in symmetrize
  constexpr int L = ld<LDN>();
  using Rw = Rows<M, NC>;
  const Rw w;
  const int i0 = w.i0 < Rw::per ? w.i0 : 0;
  const R* a = TR ? A + w.j * L + i0 : A + i0 * L + w.j;
  constexpr int step = TR ? Rw::per : Rw::per * L;
  R v[Rw::passes];
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r) v[r] = a[(w.live(r) ? r : 0) * step];
  R* o = B + i0 * L + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) o[r * Rw::per * L] = v[r];
  wsync();
}

template <int LDN, int M, int NC, typename R>
PKS_DEV void zero(R* A) {
  using Rw = Rows<M, NC>;
  const Rw w;
  R* o = A + w.i0 * ld<LDN>() + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) o[r * Rw::per * ld<LDN>()] = R(0);
  wsync();
}

// B <- A - B
template <int LDN, int M, int NC, typename R>
PKS_DEV void rsub(const R* A, R* B) {
  using Rw = Rows<M, NC>;
  const Rw w;
  const int o = (w.i0 < Rw::per ? w.i0 : 0) * ld<LDN>() + w.j;
  R v[Rw::passes];
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r) {
    const int q = (w.live(r) ? r : 0) * Rw::per * ld<LDN>();
    v[r] = A[o + q] - B[o + q];
  }
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) B[o + r * Rw::per * ld<LDN>()] = v[r];
  wsync();
}

template <int N, typename R>
PKS_DEV void vcopy(const R* x, R* y) {
  for (int i = lane(); i < N; i += kWave) y[i] = x[i];
  wsync();
}

// --- HBM <-> LDS ------------------------------------------------------------
// The element type in HBM (RG) may differ from the one in LDS (R): the FP32
// engine's linearisation works in FP64 on its FP32 records.
// All global loads are issued before the first LDS store, so one record costs
// one memory latency, not one per pass.
template <int LDN, int M, int NC, bool ADD, typename RG, typename R>
PKS_DEV void ld_rows(const RG* g, R* A) {
  using Rw = Rows<M, NC>;
  const Rw w;
  const RG* p = g + (w.i0 < Rw::per ? w.i0 : 0) * NC + w.j;
  R v[Rw::passes];
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r) v[r] = R(p[(w.live(r) ? r : 0) * Rw::per * NC]);
  R* o = A + w.i0 * ld<LDN>() + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) {
      R& x = o[r * Rw::per * ld<LDN>()];
      x = ADD ? x + v[r] : v[r];
    }
}
template <int LDN, int M, int NC, typename RG, typename R>
PKS_DEV void ld_full(const RG* g, R* A) { ld_rows<LDN, M, NC, false>(g, A); }
// A += g (row-major M x NC in HBM)
template <int LDN, int M, int NC, typename RG, typename R>
PKS_DEV void add_full(const RG* g, R* A) { ld_rows<LDN, M, NC, true>(g, A); }
template <int LDN, int M, int NC, typename R, typename RG>
PKS_DEV void st_full(const R* A, RG* g) {
  using Rw = Rows<M, NC>;
  const Rw w;
  const R* a = A + w.i0 * ld<LDN>() + w.j;
  RG* p = g + w.i0 * NC + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) p[r * Rw::per * NC] = RG(a[r * Rw::per * ld<LDN>()]);
}
template <int LDN, int N, typename RG, typename R>
PKS_DEV void ld_symm(const RG* g, R* A) {
  using Rw = Rows<N, N>;
  const Rw w;
  R v[Rw::passes];
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    v[r] = R(g[w.live(r) ? sym_index<N>(w.i0 + r * Rw::per, w.j) : 0]);
  R* o = A + w.i0 * ld<LDN>() + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r)
    if (w.live(r)) o[r * Rw::per * ld<LDN>()] = v[r];
}
template <int LDN, int N, typename R, typename RG>
PKS_DEV void st_symm(const R* A, RG* g) {
  using Rw = Rows<N, N>;
  const Rw w;
  const R* a = A + w.i0 * ld<LDN>() + w.j;
  PKS_UNROLL for (int r = 0; r < Rw::passes; ++r) {
    const int i = w.i0 + r * Rw::per;
    if (w.live(r) && w.j >= i) g[sym_index<N>(i, w.j)] = RG(a[r * Rw::per * ld<LDN>()]);
  }
}
template <int N, typename RG, typename R>
PKS_DEV void ld_v(const RG* g, R* x) {
  for (int i = lane(); i < N; i += kWave) x[i] = R(g[i]);
}
template <int N, typename R, typename RG>
PKS_DEV void st_v(const R* x, RG* g) {
  for (int i = lane(); i < N; i += kWave) g[i] = RG(x[i]);
}

// ---------------------------------------------------------------------------
// Record layouts (words of one slot, contiguous in HBM).
// ---------------------------------------------------------------------------
template <int N, int P>
struct Layout {
  static constexpr int kS = sym_size<N>(), kSP = sym_size<P>();
  static constexpr int kTraj = N + kS;                     // mean, cov
  static constexpr int kTrans = N * N + N + kS;            // F, c, Q'
  static constexpr int kHlin = P * N + P + kSP + P;        // H, d, R', ytilde
  static constexpr int kFElem = N * N + 2 * N + 2 * kS;    // A, b, C, eta, J
  static constexpr int kSElem = N * N + N + kS;            // E, g, L
  static constexpr int kCarry = N + kS;                    // (b, C) or (g, L)
  static_assert(kSElem <= kFElem, "smoothing elements reuse the filtering element records");
};

// LDS work area of one wave: NM matrices of N x N (names per kernel), sized
// per kernel so that light kernels keep more waves resident.
template <int N, typename R, int NM>
struct Work {
  static constexpr int MW = mat_words<N>();
  static constexpr int kNM = NM;
  R m[NM][MW];
  R v[8][N];       // vectors
  int ok;
};

// --- restarts -------------------------------------------------------------
// A right operand with A = 0 (filtering) or E = 0 (smoothing) -- a track's
// prior or end element, or an aggregate that contains one -- yields its own
// (b, C) resp. (g, L) whatever the left operand holds.  The formulas give that
// for finite operands; when a failed left operand has turned the result into
// NaN (0 * NaN), the restart is taken as is, so a failed track never spills
// into the tracks after it.  Every lane reads the same LDS words, so the
// branch is uniform; finite results are unchanged bit for bit.
template <int N, typename R>
PKS_DEV bool all_zero(const R* A) {
  bool z = true;
  for (int e = lane(); e < N * N; e += kWave) z = z && A[(e / N) * ld<N>() + e % N] == R(0);
  return __all(z);
}

template <int N, typename R>
PKS_DEV void take_restart(const R* rA, const R* rb, const R* rC, R* lA, R* lb, R* lC) {
  constexpr int L = ld<N>();
  for (int e = lane(); e < N * N; e += kWave) {
    const int i = e / N, j = e - i * N;
    if (lA) lA[i * L + j] = R(0);
    lC[i * L + j] = rC[i * L + j];
  }
  for (int i = lane(); i < N; i += kWave) lb[i] = rb[i];
  wsync();
}

// S = I + U^T J U (S may be J) and v = e - J b; T is scratch.
template <int N, typename R>
PKS_DEV void gain_matrix(const R* U, const R* b, const R* e, const R* J, R* S, R* T, R* v) {
  constexpr const R* none = nullptr;
  mm<N, N, N, N, false, false>(J, U, none, R(1), T, b, e, R(-1), v);   // J U
  mm<N, N, N, N, true, false>(U, T, none, R(1), S);
  for (int i = lane(); i < N; i += kWave) S[i * ld<N>() + i] += R(1);
  wsync();
}

// C = U U^T (in place: C becomes U), G = I + U^T J U (in S, which may be J) =
// Lg Lg^T and W = Lg^-1 U^T (in T); v = e - J b.  One copy of the
// factorisation serves both matrices: it is straight-line code of 9 KB, and
// two CUs share 64 KB of instruction cache.
template <int N, typename R>
PKS_DEV void gain_factors(R* C, const R* b, const R* e, const R* J, R* S, R* T, R* v, int* ok) {
  Factor<N, R> f;
#pragma unroll 1
  for (int ph = 0; ph < 2; ++ph) {
    if (ph == 1) gain_matrix<N>(C, b, e, J, S, T, v);
    chol<N, N>(ph == 0 ? C : S, ok, f, ph == 0);
  }
  fwd_t<N>(f, C, T);
}

// --- the filtering operator (eq. 15), symmetric pivot-free form ------------
// l <- l (x) r with l = (lA, lb, lC, le, lJ), r = (rA, rb, C_j, re, rJ).  Same
// algebra as FilterOp::combine.  l's C holds its Cholesky factor and then M
// while the result is formed, S holds G, its factor and Y, rJ holds A_j M (rJ
// and S are destroyed), T is scratch.  C_j enters only the last step:
// getC(S) returns it as an LDS operand (it may read it into S, free by then).
template <int N, typename R, class GetC>
PKS_DEV void combine_f_impl(R* lA, R* lb, R* lC, R* le, R* lJ, const R* rA, const R* rb, const R* re, R* rJ, R* S,
                            R* T, R* v1, R* v2, int* ok, GetC getC) {
  constexpr const R* none = nullptr;
  gain_factors<N>(lC, lb, re, rJ, S, T, v1, ok);         // lC = U, T = W, v1 = v
  mm<N, N, N, N, true, false>(T, T, (const R*)nullptr, R(1), lC);        // M = W^T W
  mm<N, N, N, N, false, false>(rJ, lA, (const R*)nullptr, R(1), S);      // Y = J A_i
  mm<N, N, N, N, false, false>(lC, S, none, R(1), T, v1, none, R(1), v2);  // Z = M Y; u = M v
  // J_ij = A_i^T Y - Y^T Z + J_i ; eta_ij = A_i^T v - Y^T u + eta_i
  mm<N, N, N, N, true, false>(lA, S, lJ, R(1), lJ, v1, le, R(1), le);
  mm<N, N, N, N, true, false>(S, T, lJ, R(-1), lJ, v2, le, R(-1), le);
  symmetrize<N, N>(lJ);
  // b_ij = A_j (b_i + u) + b_j
  for (int i = lane(); i < N; i += kWave) v1[i] = lb[i] + v2[i];
  wsync();
  // C_ij = A_j M A_j^T + C_j
  mm<N, N, N, N, false, false>(rA, lC, none, R(1), rJ, v1, rb, R(1), lb);  // A_j M
  const R* rC = getC(S);
  mm<N, N, N, N, false, true>(rJ, rA, rC, R(1), lC);
  symmetrize<N, N>(lC);
  // A_ij = A_j (A_i - Z)
  rsub<N, N, N>(lA, T);
  mm<N, N, N, N, false, false>(rA, T, (const R*)nullptr, R(1), lA);
  if (!(lb[0] == lb[0]) && all_zero<N>(rA)) take_restart<N>(rA, rb, rC, lA, lb, lC);
}

// All operands in LDS; S and T scratch, rJ destroyed.  The routine-cycle probe
// times this form.
template <int N, typename R>
PKS_DEV void combine_f(R* lA, R* lb, R* lC, R* le, R* lJ, const R* rA, const R* rb, const R* rC, const R* re, R* rJ,
                       R* S, R* T, R* v1, R* v2, int* ok) {
  combine_f_impl<N, R>(lA, lb, lC, le, lJ, rA, rb, re, rJ, S, T, v1, v2, ok, [&](R*) { return rC; });
}

// The kernels' form: C_j stays in the right element's record in global memory
// (gC, symmetric packed, written before the call) and is read into rC, which
// serves as S until then; the right element takes two LDS matrices (rA, rJ)
// plus rC, and the call one scratch matrix T.
template <int N, typename R, typename RG>
PKS_DEV void combine_f_lean(R* lA, R* lb, R* lC, R* le, R* lJ, const R* rA, const R* rb, R* rC, const R* re,
                            R* rJ, const RG* gC, R* T, R* v1, R* v2, int* ok) {
  combine_f_impl<N, R>(lA, lb, lC, le, lJ, rA, rb, re, rJ, rC, T, v1, v2, ok, [&](R* buf) {
    ld_symm<N, N>(gC, buf);
    wsync();
    return static_cast<const R*>(buf);
  });
}

// The carry application after gain_factors: from T = W and v1 = v.
template <int N, typename R, class GetC>
PKS_DEV void apply_gain(R* cb, R* cC, const R* rA, const R* rb, R* rJ, R* T, R* v1, R* v2, GetC getC) {
  constexpr const R* none = nullptr;
  mm<N, N, N, N, true, false>(T, T, (const R*)nullptr, R(1), cC);        // M = W^T W
  mv<N, N, N, false>(cC, v1, (const R*)nullptr, R(1), v2);               // u = M v
  for (int i = lane(); i < N; i += kWave) v1[i] = cb[i] + v2[i];
  wsync();
  mm<N, N, N, N, false, false>(rA, cC, none, R(1), T, v1, rb, R(1), cb);   // A M
  const R* rC = getC(rJ);
  mm<N, N, N, N, false, true>(T, rA, rC, R(1), cC);     // A M A^T + C
  symmetrize<N, N>(cC);
  if (!(cb[0] == cb[0]) && all_zero<N>(rA)) take_restart<N>(rA, rb, rC, (R*)nullptr, cb, cC);
}

// Carry (b, C) (x) r: the filtered mean and covariance after element r.  The
// carry's covariance holds its Cholesky factor and then M while the result is
// formed, rJ holds G and its factor (rJ is destroyed), T is scratch.  The
// element's C enters only the last step: getC(rJ) returns it as an LDS
// operand (it may read it into rJ, free by then).
template <int N, typename R, class GetC>
PKS_DEV void apply_f_impl(R* cb, R* cC, const R* rA, const R* rb, const R* re, R* rJ, R* T, R* v1, R* v2, int* ok,
                          GetC getC) {
  gain_factors<N>(cC, cb, re, rJ, rJ, T, v1, ok);        // cC = U, T = W, v1 = v
  apply_gain<N, R>(cb, cC, rA, rb, rJ, T, v1, v2, getC);
}

// All operands in LDS; one scratch matrix T, rJ destroyed.
template <int N, typename R>
PKS_DEV void apply_f(R* cb, R* cC, const R* rA, const R* rb, const R* rC, const R* re, R* rJ, R* T, R* v1, R* v2,
                     int* ok) {
  apply_f_impl<N, R>(cb, cC, rA, rb, re, rJ, T, v1, v2, ok, [&](R*) { return rC; });
}

// --- the smoothing operator (eq. 19) ------------------------------------------
// l <- l (x) r in the paper's order (l earlier in time): (E_l E_r, E_l g_r + g_l, E_l L_r E_l^T + L_l).
// T1 and T2 are scratch and may be the same matrix.
template <int N, typename R>
PKS_DEV void combine_s(R* lE, R* lg, R* lL, const R* rE, const R* rg, const R* rL, R* T1, R* T2, R* v1) {
  // E_l = 0 (a track's end element or an aggregate holding one): the result
  // is l itself; l is updated in place, so the restart is taken up front.
  if (lE[0] == R(0) && all_zero<N>(lE)) return;
  constexpr const R* none = nullptr;
  mm<N, N, N, N, false, false>(lE, rL, none, R(1), T1, rg, none, R(1), v1);
  mm<N, N, N, N, false, true>(T1, lE, lL, R(1), lL);
  symmetrize<N, N>(lL);
  mm<N, N, N, N, false, false>(lE, rE, (const R*)nullptr, R(1), T2);
  copy<N, N, N, false>(T2, lE);
  for (int i = lane(); i < N; i += kWave) lg[i] += v1[i];
  wsync();
}

// r (x) carry (g, L): the smoothed mean and covariance before the carry.
template <int N, typename R>
PKS_DEV void apply_s(const R* rE, const R* rg, const R* rL, R* cg, R* cL, R* T1, R* v1) {
  mm<N, N, N, N, false, false>(rE, cL, (const R*)nullptr, R(1), T1, cg, rg, R(1), v1);
  mm<N, N, N, N, false, true>(T1, rE, rL, R(1), cL);
  symmetrize<N, N>(cL);
  vcopy<N>(v1, cg);
  if (!(cg[0] == cg[0] && cL[0] == cL[0]) && all_zero<N>(rE)) take_restart<N>(rE, rg, rL, (R*)nullptr, cg, cL);
}

// --- statistical linear regression (eq. 7-9) of g: R^N -> R^Q at (xbar, Pbar)
// with the symmetric sigma-point set of elements.hpp (slr): one sigma point
// per lane.  Inputs xbar (LDS vector) and Pbar (LDS matrix, destroyed: it
// becomes its Cholesky factor).  Outputs G (Q x N, LDS), off = zbar - G xbar,
// Lam (Q x Q), zc = g(xbar).  Zp, Zm, D: N x Q scratch; zbar: Q vector.  D may
// be Zp and G may be Zm (D is formed in place once Phi has read the images,
// G once D is done with them), so the regression fits in four matrices.
template <int N, int Q, bool kAngular, typename R, class Eval>
PKS_DEV void slr(int lin, SigmaRule rule, const R* xbar, R* Pbar, Eval eval, R* G, R* off, R* Lam, R* zc, R* Zp,
                 R* Zm, R* D, R* zbar, int* ok, bool factored = false) {
  constexpr int L = ld<N>();
  if (!factored) chol<N, N>(Pbar, ok);    // else Pbar already holds the factor
  R gamma, w0, wj;
  sigma_weights<N, R>(lin, rule, gamma, w0, wj);
  // all 2N + 1 points in one pass: lane 2N takes the centre
  static_assert(2 * N + 1 <= kWave, "one sigma point per lane");
  if (const int ln = lane(); ln <= 2 * N) {
    const bool centre = ln == 2 * N;
    const int j = ln < N ? ln : (centre ? 0 : ln - N);
    const R sg = ln < N ? gamma : -gamma;
    R x[N], z[Q];
    PKS_UNROLL for (int i = 0; i < N; ++i) x[i] = centre ? xbar[i] : xbar[i] + sg * Pbar[i * L + j];
    eval(x, z);
    R* out = centre ? zc : (ln < N ? Zp + j * L : Zm + j * L);
    PKS_UNROLL for (int q = 0; q < Q; ++q) out[q] = z[q];
  }
  wsync();
  if constexpr (kAngular) {   // each image on the branch of the centre's
    for (int e = lane(); e < 2 * N * Q; e += kWave) {
      const int jj = e / Q, q = e - jj * Q;
      R* v = (jj < N ? Zp + jj * L : Zm + (jj - N) * L) + q;
      *v = zc[q] + wrap_pi<R>(*v - zc[q]);
    }
    wsync();
  }
  for (int q = lane(); q < Q; q += kWave) {
    R s = R(0);
    for (int j = 0; j < N; ++j) s += Zp[j * L + q] + Zm[j * L + q];
    zbar[q] = w0 * zc[q] + wj * s;
  }
  wsync();
  // Lambda = Phi - D^T D, Phi = sum_j w_j (Z_j - zbar)(Z_j - zbar)^T
  const R wg = wj * gamma;
  auto form_D = [&] {
    for (int e = lane(); e < N * Q; e += kWave) {
      const int j = e / Q, q = e - j * Q;
      D[j * L + q] = wg * (Zp[j * L + q] - Zm[j * L + q]);
    }
    wsync();
  };
  if constexpr (Q * Q > kWave && Q % 2 == 0 && (Q / 2) * (Q / 2 + 1) / 2 <= kWave) {
    // a 2 x 2 tile of the upper triangle per lane (Q = 20: 55 tiles, one
    // round), each entry summed in the order and with the roundings of the
    // one-entry loops below.  With one entry per lane the two sums took seven
    // rounds over 400 entries, half of them below the diagonal, and each
    // operand was read from LDS for one product: the kernel, bound by its
    // instructions, took 947 us for 65,537 slots and takes 716 us.
    constexpr int T = Q / 2;
    const int t = lane();
    int ta = 0;
    PKS_UNROLL for (int k = 1; k < T; ++k) ta += t >= k * T - k * (k - 1) / 2;
    const bool live = t < T * (T + 1) / 2;
    const int a0 = live ? 2 * ta : 0, b0 = live ? 2 * (t - (ta * T - ta * (ta - 1) / 2) + ta) : 0;
    const R za[2] = {zbar[a0], zbar[a0 + 1]}, zb[2] = {zbar[b0], zbar[b0 + 1]};
    R s[2][2] = {{R(0), R(0)}, {R(0), R(0)}};
#pragma unroll 2
    for (int j = 0; j < N; ++j) {
      const R *p = Zp + j * L, *m = Zm + j * L;
      R pa[2], pb[2], ma[2], mb[2];
      PKS_UNROLL for (int i = 0; i < 2; ++i) {
        pa[i] = p[a0 + i] - za[i];
        pb[i] = p[b0 + i] - zb[i];
        ma[i] = m[a0 + i] - za[i];
        mb[i] = m[b0 + i] - zb[i];
      }
      PKS_UNROLL for (int i = 0; i < 2; ++i)
        PKS_UNROLL for (int k = 0; k < 2; ++k) s[i][k] += fma(pa[i], pb[k], ma[i] * mb[k]);
    }
    PKS_UNROLL for (int i = 0; i < 2; ++i)
      PKS_UNROLL for (int k = 0; k < 2; ++k)
        s[i][k] = fma(w0 * (zc[a0 + i] - za[i]), zc[b0 + k] - zb[k], s[i][k] * wj);
    wsync();
    form_D();
#pragma unroll 4
    for (int j = 0; j < N; ++j) {
      const R* d = D + j * L;
      PKS_UNROLL for (int i = 0; i < 2; ++i) PKS_UNROLL for (int k = 0; k < 2; ++k) s[i][k] -= d[a0 + i] * d[b0 + k];
    }
    if (live) {
      PKS_UNROLL for (int i = 0; i < 2; ++i)
        PKS_UNROLL for (int k = 0; k < 2; ++k) {
          if (i == 1 && k == 0 && a0 == b0) continue;   // below the diagonal of a diagonal tile
          Lam[(a0 + i) * L + b0 + k] = s[i][k];
          Lam[(b0 + k) * L + a0 + i] = s[i][k];
        }
    }
    wsync();
  } else {
    for (int e = lane(); e < Q * Q; e += kWave) {
      const int a = e / Q, b = e - a * Q;
      if (b < a) continue;
      R s = R(0);
      for (int j = 0; j < N; ++j)
        s += (Zp[j * L + a] - zbar[a]) * (Zp[j * L + b] - zbar[b]) +
             (Zm[j * L + a] - zbar[a]) * (Zm[j * L + b] - zbar[b]);
      s = s * wj + w0 * (zc[a] - zbar[a]) * (zc[b] - zbar[b]);
      Lam[a * L + b] = s;
    }
    wsync();
    form_D();
    for (int e = lane(); e < Q * Q; e += kWave) {
      const int a = e / Q, b = e - a * Q;
      if (b < a) continue;
      R s = Lam[a * L + b];
      for (int j = 0; j < N; ++j) s -= D[j * L + a] * D[j * L + b];
      Lam[a * L + b] = s;
      Lam[b * L + a] = s;
    }
    wsync();
  }
  bwd<N, N, Q>(Pbar, D);                    // G^T = L^-T D
  copy<N, Q, N, true>(D, G);
  for (int q = lane(); q < Q; q += kWave) {
    R s = zbar[q];
    for (int i = 0; i < N; ++i) s -= G[q * L + i] * xbar[i];
    off[q] = s;
  }
  wsync();
}

// ---------------------------------------------------------------------------
// Kernel arguments.
// ---------------------------------------------------------------------------
struct DnArgs {
  int64_t S;
  int ntracks;
  int lin;
  SigmaRule rule;
  const unsigned char* flags;   // kSlotFirst / kSlotLast per slot
  const int* track;             // track of each slot
  const void* params;
  const void* Q;                // N x N full
  const void* Rm;               // P x P full
  const double* params64;       // the same three in FP64, for the linearisation
  const double* Q64;
  const double* Rm64;
  const void* m0;               // [track][N]
  const void* P0;               // [track][N][N] full
  const void* y;                // [slot][P] (slot 0 of a track unused)
  void* traj;                   // [slot][kTraj]
  void* trans;                  // [slot][kTrans]
  void* hlin;                   // [slot][kHlin]
  void* elem;                   // [slot][kFElem]; smoothing elements reuse it
  unsigned long long* delta_bits;
  double lm;                    // Levenberg-Marquardt damping lambda (0 = undamped)
};

// The same model in another precision (model templates are <N, P, real>).
template <class M, typename T>
struct WithReal;
template <template <int, int, typename> class Mt, int N, int P, typename R, typename T>
struct WithReal<Mt<N, P, R>, T> {
  using type = Mt<N, P, T>;
};

struct DnLevel {
  const void* in;    // aggregates of this level (count n)
  void* out;         // aggregates of the next level (count ceil(n / fan))
  void* carry_out;   // exclusive carries of this level's elements (count n)
  const void* carry_in;  // exclusive carries of the next level's chunks
  int64_t n;
  int fan;
};

template <class Model, typename R>
struct Dense {
  static constexpr int N = Model::N, P = Model::P;
  using Lay = Layout<N, P>;
  using W = Work<N, R, 9>;
  template <int NM>
  using WorkN = Work<N, R, NM>;

  // element a_s into (A, b, C, eta, J) in the given LDS buffers, with one
  // scratch matrix T: F and Q' are read into A's and C's buffers (A and C are
  // formed over them), S and H into rows 0..P-1 and P..2P-1 of J's buffer (J
  // is formed last), H Q' and H F into the same rows of T.  A work area of
  // nine matrices also takes the Levenberg-Marquardt damping (w.m[6..8]).
  template <class WT>
  static PKS_DEV void build_element(const DnArgs& a, int64_t s, WT& w, R* T, R* A, R* b, R* C, R* e, R* J) {
    static_assert(2 * P <= N, "S and H share one matrix buffer");
    constexpr int L = ld<N>();
    const unsigned fl = a.flags[s];
    if (fl & kSlotFirst) {
      const int tr = a.track[s];
      zero<N, N, N>(A);
      zero<N, N, N>(J);
      ld_v<N>(static_cast<const R*>(a.m0) + size_t(tr) * N, b);
      ld_full<N, N, N>(static_cast<const R*>(a.P0) + size_t(tr) * N * N, C);
      for (int i = lane(); i < N; i += kWave) e[i] = R(0);
      wsync();
      if constexpr (WT::kNM >= 9) {
        if (a.lm > 0.0) lm_damp(a, s, w, A, b, C, e, J);
      }
      return;
    }
    // transition out of slot s - 1, measurement at slot s
    const R* tr = static_cast<const R*>(a.trans) + size_t(s - 1) * Lay::kTrans;
    const R* hl = static_cast<const R*>(a.hlin) + size_t(s) * Lay::kHlin;
    R* F = A;
    R* Qp = C;
    R* Sx = J;          // P x P
    R* H = J + P * L;   // P x N
    R* c = w.v[4];
    R* d = w.v[5];
    R* yt = w.v[6];
    ld_full<N, N, N>(tr, F);
    ld_v<N>(tr + N * N, c);
    ld_symm<N, N>(tr + N * N + N, Qp);
    ld_full<N, P, N>(hl, H);
    ld_v<P>(hl + P * N, d);
    ld_symm<N, P>(hl + P * N + P, Sx);
    ld_v<P>(hl + P * N + P + Lay::kSP, yt);
    wsync();
    R* HQ = T;          // P x N
    R* HF = T + P * L;  // P x N
    mm<N, P, N, N, false, false>(H, Qp, (const R*)nullptr, R(1), HQ);
    mm<N, P, N, N, false, false>(H, F, (const R*)nullptr, R(1), HF, c, yt, R(-1), yt);   // w = y - H c - d
    mm<N, P, N, P, false, true>(HQ, H, Sx, R(1), Sx);                      // S = H Q' H^T + R'
    for (int i = lane(); i < P; i += kWave) yt[i] -= d[i];
    wsync();
    {
      Factor<P, R> Ls;
      chol<N, P>(Sx, &w.ok, Ls, false);
      fwd2<N, N>(Ls, HQ, HF, yt);                     // Zs = Ls^-1 H Q', Ys = Ls^-1 H F, ws = Ls^-1 w
    }
    mm<N, N, P, N, true, false>(HQ, HF, F, R(-1), A, yt, c, R(1), b);       // A = F - Zs^T Ys, b = c + Zs^T ws
    mm<N, N, P, N, true, false>(HQ, HQ, Qp, R(-1), C);                      // C = Q' - Zs^T Zs
    mm<N, N, P, N, true, false>(HF, HF, (const R*)nullptr, R(1), J, yt, (const R*)nullptr, R(1), e);
                                                                            // J = Ys^T Ys, eta = Ys^T ws
    symmetrize<N, N>(C);
    symmetrize<N, N>(J);
    if constexpr (WT::kNM >= 9) {
      if (a.lm > 0.0) lm_damp(a, s, w, A, b, C, e, J);
    }
  }

  // Levenberg-Marquardt damping of the element of slot s (Section 3, damped
  // Gauss-Newton extension): the previous iterate xbar_s is observed through
  // x_s with noise covariance I/lambda.  With G = I + lambda C = L L^T,
  // Z = L^-1 C, V = L^-1 A, v = L^-1 (xbar - b):
  //   A -= lambda Z^T V,  b += lambda Z^T v,  C -= lambda Z^T Z,
  //   J += lambda V^T V,  eta += lambda V^T v.
  // Scratch: w.m[6..8], w.v[4] (free once the element is built).
  template <class WT>
  static PKS_DEV void lm_damp(const DnArgs& a, int64_t s, WT& w, R* A, R* b, R* C, R* e, R* J) {
    constexpr int L = ld<N>();
    const R lam = R(a.lm);
    const R* xbar = static_cast<const R*>(a.traj) + size_t(s) * Lay::kTraj;
    R* G = w.m[6];
    R* Z = w.m[7];
    R* V = w.m[8];
    R* v = w.v[4];
    for (int t = lane(); t < N * N; t += kWave) {
      const int i = t / N, j = t - i * N;
      G[i * L + j] = lam * C[i * L + j] + (i == j ? R(1) : R(0));
      Z[i * L + j] = C[i * L + j];
      V[i * L + j] = A[i * L + j];
    }
    for (int i = lane(); i < N; i += kWave) v[i] = xbar[i] - b[i];
    wsync();
    {
      Factor<N, R> Lg;
      chol<N, N>(G, &w.ok, Lg, false);
      fwd2<N, N>(Lg, Z, V, v);
    }
    mv<N, N, N, true>(Z, v, b, lam, b);
    mv<N, N, N, true>(V, v, e, lam, e);
    mm<N, N, N, N, true, false>(Z, V, A, -lam, A);
    mm<N, N, N, N, true, false>(Z, Z, C, -lam, C);
    mm<N, N, N, N, true, false>(V, V, J, lam, J);
    symmetrize<N, N>(C);
    symmetrize<N, N>(J);
  }

  static PKS_DEV void store_felem(const R* A, const R* b, const R* C, const R* e, const R* J, R* g) {
    st_full<N, N, N>(A, g);
    st_v<N>(b, g + N * N);
    st_symm<N, N>(C, g + N * N + N);
    st_v<N>(e, g + N * N + N + Lay::kS);
    st_symm<N, N>(J, g + N * N + 2 * N + Lay::kS);
  }
  static PKS_DEV void load_felem(const R* g, R* A, R* b, R* C, R* e, R* J) {
    ld_full<N, N, N>(g, A);
    ld_v<N>(g + N * N, b);
    ld_symm<N, N>(g + N * N + N, C);
    ld_v<N>(g + N * N + N + Lay::kS, e);
    ld_symm<N, N>(g + N * N + 2 * N + Lay::kS, J);
    wsync();
  }
  static PKS_DEV void store_selem(const R* E, const R* g_, const R* Lm, R* g) {
    st_full<N, N, N>(E, g);
    st_v<N>(g_, g + N * N);
    st_symm<N, N>(Lm, g + N * N + N);
  }
  static PKS_DEV void load_selem(const R* g, R* E, R* g_, R* Lm) {
    ld_full<N, N, N>(g, E);
    ld_v<N>(g + N * N, g_);
    ld_symm<N, N>(g + N * N + N, Lm);
    wsync();
  }
  static PKS_DEV void store_carry(const R* x, const R* Pm, R* g) {
    st_v<N>(x, g);
    st_symm<N, N>(Pm, g + N);
  }
  static PKS_DEV void load_carry(const R* g, R* x, R* Pm) {
    ld_v<N>(g, x);
    ld_symm<N, N>(g + N, Pm);
    wsync();
  }
};

// ---------------------------------------------------------------------------
// Kernels.  Every workgroup is one wave (64 lanes).
// ---------------------------------------------------------------------------

// Linearisation of f (all but the last slot of a track) and h (all but the
// first) at the current trajectory; one slot per workgroup.
template <class Model, typename R>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(3))) void k_dn_linearize(DnArgs a) {
  // The regression runs in FP64 whatever the records' type R: in FP32 its
  // sums of sigma-point images (z-bar - G x-bar, Phi - D^T D) would cost more
  // accuracy than the FP32 scan itself.
  using RC = double;
  using MC = typename WithReal<Model, RC>::type;
  using D = Dense<MC, RC>;
  constexpr int N = D::N, P = D::P;
  using Lay = typename D::Lay;
  __shared__ typename D::template WorkN<4> w;   // Pbar's factor; images and D; images and G; Lambda
  const int64_t s = blockIdx.x;
  if (s >= a.S) return;
  if (lane() == 0) w.ok = 1;
  const MC md{a.params64};
  const unsigned fl = a.flags[s];
  const R* tj = static_cast<const R*>(a.traj) + size_t(s) * Lay::kTraj;
  RC* xbar = w.v[0];
  ld_v<N>(tj, xbar);
  wsync();
  bool factored = false;   // w.m[0] holds the Cholesky factor of Pbar, shared by f and h
  if (!(fl & kSlotLast)) {
    ld_symm<N, N>(tj + N, w.m[0]);
    wsync();
    RC* G = w.m[2];
    RC* Lam = w.m[3];
    slr<N, N, false, RC>(a.lin, a.rule, xbar, w.m[0], [&](const RC(&x)[N], RC(&z)[N]) { md.f(x, z); }, G, w.v[1],
                         Lam, w.v[2], w.m[1], w.m[2], w.m[1], w.v[3], &w.ok);
    factored = true;
    R* out = static_cast<R*>(a.trans) + size_t(s) * Lay::kTrans;
    add_full<N, N, N>(a.Q64, Lam);
    wsync();
    st_full<N, N, N>(G, out);
    st_v<N>(w.v[1], out + N * N);
    st_symm<N, N>(Lam, out + N * N + N);
    wsync();                      // the stores have read LDS before it is reused
  }
  if (!(fl & kSlotFirst)) {
    if (!factored) {
      ld_symm<N, N>(tj + N, w.m[0]);
      wsync();
    }
    RC* H = w.m[2];
    RC* Om = w.m[3];
    RC* hc = w.v[2];
    slr<N, P, MC::kAngular, RC>(a.lin, a.rule, xbar, w.m[0], [&](const RC(&x)[N], RC(&z)[P]) { md.h(x, z); }, H,
                                w.v[1], Om, hc, w.m[1], w.m[2], w.m[1], w.v[3], &w.ok, factored);
    R* out = static_cast<R*>(a.hlin) + size_t(s) * Lay::kHlin;
    const R* y = static_cast<const R*>(a.y) + size_t(s) * P;
    add_full<N, P, P>(a.Rm64, Om);
    for (int i = lane(); i < P; i += kWave)
      out[P * N + P + Lay::kSP + i] = R(MC::kAngular ? hc[i] + wrap_pi<RC>(RC(y[i]) - hc[i]) : RC(y[i]));
    wsync();
    st_full<N, P, N>(H, out);
    st_v<P>(w.v[1], out + P * N);
    st_symm<N, P>(Om, out + P * N + P);
  }
}

// Level 0 of the filtering scan: build the elements of `fan` consecutive
// slots, store them, and fold them into the chunk aggregate.  The aggregate,
// the element being folded in and one scratch matrix take seven matrices
// (24.8 KB in FP64: six waves per CU); the damped form (kDamp, lambda > 0)
// has two more for the damping.
template <class Model, typename R, bool kDamp>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 3 : 2))) void k_dn_forward_up(DnArgs a, int fan, void* agg_out) {
  using D = Dense<Model, R>;
  constexpr int N = D::N;
  using Lay = typename D::Lay;
  __shared__ typename D::template WorkN<kDamp ? 9 : 7> w;
  if (lane() == 0) w.ok = 1;
  const int64_t s0 = int64_t(blockIdx.x) * fan;
  const int64_t s1 = min(s0 + fan, a.S);
  R *lA = w.m[0], *lC = w.m[1], *lJ = w.m[2], *rA = w.m[3], *rJ = w.m[4], *rC = w.m[5], *T = w.m[6];
  R *lb = w.v[0], *le = w.v[1], *rb = w.v[2], *re = w.v[3];
  for (int64_t s = s0; s < s1; ++s) {
    R* A = s == s0 ? lA : rA;
    R* C = s == s0 ? lC : rC;
    R* J = s == s0 ? lJ : rJ;
    R* b = s == s0 ? lb : rb;
    R* e = s == s0 ? le : re;
    R* rec = static_cast<R*>(a.elem) + size_t(s) * Lay::kFElem;
    D::build_element(a, s, w, T, A, b, C, e, J);
    D::store_felem(A, b, C, e, J, rec);
    if (s > s0)
      combine_f_lean<N, R>(lA, lb, lC, le, lJ, rA, rb, rC, re, rJ, rec + N * N + N, T, w.v[4], w.v[5], &w.ok);
  }
  D::store_felem(lA, lb, lC, le, lJ, static_cast<R*>(agg_out) + size_t(blockIdx.x) * Lay::kFElem);
}

// Up-sweep of a scan level: fold `fan` consecutive aggregates.  FILT selects
// the operator (filtering: records of kFElem words; smoothing: kSElem).
template <class Model, bool FILT, typename R>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_dn_scan_up(DnArgs a, DnLevel lv) {
  using D = Dense<Model, R>;
  constexpr int N = D::N;
  using Lay = typename D::Lay;
  constexpr int RW = FILT ? Lay::kFElem : Lay::kSElem;
  __shared__ typename D::template WorkN<FILT ? 7 : 6> w;
  if (lane() == 0) w.ok = 1;
  const int64_t i0 = int64_t(blockIdx.x) * lv.fan;
  const int64_t i1 = min(i0 + lv.fan, lv.n);
  const R* in = static_cast<const R*>(lv.in);
  R* out = static_cast<R*>(lv.out) + size_t(blockIdx.x) * RW;
  if (FILT) {
    D::load_felem(in + size_t(i0) * RW, w.m[0], w.v[0], w.m[1], w.v[1], w.m[2]);
    for (int64_t i = i0 + 1; i < i1; ++i) {
      // the right operand's C stays in its record until the combine's last step
      const R* g = in + size_t(i) * RW;
      ld_full<N, N, N>(g, w.m[3]);
      ld_v<N>(g + N * N, w.v[2]);
      ld_v<N>(g + N * N + N + Lay::kS, w.v[3]);
      ld_symm<N, N>(g + N * N + 2 * N + Lay::kS, w.m[5]);
      wsync();
      combine_f_lean<N, R>(w.m[0], w.v[0], w.m[1], w.v[1], w.m[2], w.m[3], w.v[2], w.m[4], w.v[3], w.m[5],
                           g + N * N + N, w.m[6], w.v[4], w.v[5], &w.ok);
    }
    D::store_felem(w.m[0], w.v[0], w.m[1], w.v[1], w.m[2], out);
  } else {
    D::load_selem(in + size_t(i0) * RW, w.m[0], w.v[0], w.m[1]);
    for (int64_t i = i0 + 1; i < i1; ++i) {
      D::load_selem(in + size_t(i) * RW, w.m[2], w.v[1], w.m[3]);
      combine_s<N, R>(w.m[0], w.v[0], w.m[1], w.m[2], w.v[1], w.m[3], w.m[4], w.m[5], w.v[2]);
    }
    D::store_selem(w.m[0], w.v[0], w.m[1], out);
  }
}

// Down-sweep of a scan level: exclusive carries of the `fan` aggregates of one
// chunk from the chunk's own exclusive carry.  Filtering runs forward (the
// first element overall has no carry: it starts at a prior element);
// smoothing runs backward (the last element overall has none: it ends at a
// last slot).
template <class Model, bool FILT, typename R>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_dn_scan_down(DnArgs a, DnLevel lv) {
  using D = Dense<Model, R>;
  constexpr int N = D::N;
  using Lay = typename D::Lay;
  constexpr int RW = FILT ? Lay::kFElem : Lay::kSElem;
  __shared__ typename D::template WorkN<5> w;
  if (lane() == 0) w.ok = 1;
  const int64_t c = blockIdx.x;
  const int64_t i0 = c * lv.fan;
  const int64_t i1 = min(i0 + lv.fan, lv.n);
  const int64_t nchunks = (lv.n + lv.fan - 1) / lv.fan;
  const R* in = static_cast<const R*>(lv.in);
  R* cout = static_cast<R*>(lv.carry_out);
  R *cx = w.v[6], *cP = w.m[4];
  R *rA = w.m[0], *rC = w.m[1], *rJ = w.m[2], *rb = w.v[0], *re = w.v[1];
  bool have = FILT ? c > 0 : c < nchunks - 1;
  if (have) D::load_carry(static_cast<const R*>(lv.carry_in) + size_t(c) * Lay::kCarry, cx, cP);
  for (int64_t k = 0; k < i1 - i0; ++k) {
    const int64_t i = FILT ? i0 + k : i1 - 1 - k;
    if (have) {
      D::store_carry(cx, cP, cout + size_t(i) * Lay::kCarry);
      wsync();
    }
    if (k + 1 == i1 - i0) break;   // the carry past the chunk's last aggregate is not needed
    if (FILT) {
      D::load_felem(in + size_t(i) * RW, rA, rb, rC, re, rJ);
      if (have) {
        apply_f<N, R>(cx, cP, rA, rb, rC, re, rJ, w.m[3], w.v[2], w.v[3], &w.ok);
      } else {
        vcopy<N>(rb, cx);
        copy<N, N, N, false>(rC, cP);
      }
    } else {
      D::load_selem(in + size_t(i) * RW, rA, rb, rC);
      if (have) {
        apply_s<N, R>(rA, rb, rC, cx, cP, w.m[3], w.v[2]);
      } else {
        vcopy<N>(rb, cx);
        copy<N, N, N, false>(rC, cP);
      }
    }
    have = true;
  }
}

// Level 0 down-sweep of the filtering scan and level 0 up-sweep of the
// smoothing scan: filtered x*, P* of every slot of the chunk, its smoothing
// element (eq. 17-18, stored over the filtering element) and the chunk's
// smoothing aggregate.
template <class Model, typename R>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 4 ? 3 : 2))) void k_dn_forward_down_backward_up(DnArgs a, int fan, const void* carry_in,
                                                                       void* sagg_out) {
  using D = Dense<Model, R>;
  constexpr int N = D::N;
  using Lay = typename D::Lay;
  constexpr int L = ld<N>();
  __shared__ typename D::template WorkN<6> w;
  if (lane() == 0) w.ok = 1;
  const int64_t c = blockIdx.x;
  const int64_t s0 = c * fan;
  const int64_t s1 = min(s0 + fan, a.S);
  R *cx = w.v[6], *cP = w.m[3];                       // filtered mean / covariance (carry)
  R *rA = w.m[0], *rJ = w.m[1], *T = w.m[2], *rb = w.v[0], *re = w.v[1];
  R *sE = w.m[4], *sL = w.m[5], *sg = w.v[7];          // smoothing aggregate
  bool have = c > 0;
  if (have) D::load_carry(static_cast<const R*>(carry_in) + size_t(c) * Lay::kCarry, cx, cP);
  for (int64_t s = s0; s < s1; ++s) {
    R* rec = static_cast<R*>(a.elem) + size_t(s) * Lay::kFElem;
    const R* recC = rec + N * N + N;                   // the element's C stays in the record
    ld_full<N, N, N>(rec, rA);
    ld_v<N>(rec + N * N, rb);
    ld_v<N>(rec + N * N + N + Lay::kS, re);
    ld_symm<N, N>(rec + N * N + 2 * N + Lay::kS, rJ);
    wsync();
    const bool last = a.flags[s] & kSlotLast;
    if (!have) {
      vcopy<N>(rb, cx);
      ld_symm<N, N>(recC, cP);
      wsync();
    }
    // The carry application (the steps of gain_factors and apply_gain), then
    // the smoothing element of slot s into (eE, eg, eL) = (m[0], rb, m[1]),
    // the filtering element being spent.  Phases 0, 1 and 2 factorise P*, G
    // and P^-; one copy of the factorisation and of the substitution serves
    // them (see gain_factors).
    R *eE = w.m[0], *eg = rb, *eL = w.m[1];
    R *F = w.m[1], *Pp = w.m[0], *V = T, *v = w.v[2], *t = w.v[3];
#pragma unroll 1
    for (int ph = have ? 0 : 2; ph < (last ? 2 : 3); ++ph) {
      if (ph == 1) {
        gain_matrix<N>(cP, cx, re, rJ, rJ, T, v);
      } else if (ph == 2) {
        const R* tr = static_cast<const R*>(a.trans) + size_t(s) * Lay::kTrans;
        ld_full<N, N, N>(tr, F);
        ld_symm<N, N>(tr + N * N + N, Pp);
        ld_v<N>(tr + N * N, v);
        wsync();
        mm<N, N, N, N, false, false>(F, cP, (const R*)nullptr, R(1), V, cx, v, R(1), t);   // F P*, F x* + c
        mm<N, N, N, N, false, true>(V, F, Pp, R(1), Pp);                  // F P* F^T + Q'
        symmetrize<N, N>(Pp);
      }
      Factor<N, R> f;
      chol<N, N>(ph == 0 ? cP : (ph == 1 ? rJ : Pp), &w.ok, f, ph == 0);
      if (ph == 0) continue;
      // W = Lg^-1 U^T into T; V = Lp^-1 F P* in place, t <- Lp^-1 (F x* + c)
      const int ln = lane(), row = (ln < N ? ln : 0) * L;
      Vec<R> d = columns<N, N>(ln, T);
      if (ph == 2 && ln == N) d = Vec<R>{t, 1, true};
      const Vec<R> src = ph == 1 ? Vec<R>{cP + row, 1, false} : d;
      R x[N];
      src.get(x);
      solve_l(f, x);
      d.put(x);
      if (ph == 1) {
        wsync();
        apply_gain<N, R>(cx, cP, rA, rb, rJ, T, v, t, [&](R* buf) {
          ld_symm<N, N>(recC, buf);
          wsync();
          return static_cast<const R*>(buf);
        });
      } else {
        // E^T = Lp^-T V, stored transposed over P^-
        solve_lt(f, x);
        Vec<R>{eE + row, 1, ln < N}.put(x);
        wsync();
        // L_s = P* - V^T V, g = x* - V^T Lp^-1 (F x* + c)
        mm<N, N, N, N, true, false>(V, V, cP, R(-1), eL, t, cx, R(-1), eg);
        symmetrize<N, N>(eL);
      }
    }
    have = true;
    if (last) {
      zero<N, N, N>(eE);
      vcopy<N>(cx, eg);
      copy<N, N, N, false>(cP, eL);
    }
    D::store_selem(eE, eg, eL, rec);
    if (s == s0) {
      copy<N, N, N, false>(eE, sE);
      copy<N, N, N, false>(eL, sL);
      vcopy<N>(eg, sg);
    } else {
      combine_s<N, R>(sE, sg, sL, eE, eg, eL, T, T, w.v[2]);
    }
  }
  (void)L;
  D::store_selem(sE, sg, sL, static_cast<R*>(sagg_out) + size_t(c) * Lay::kSElem);
}

// Level 0 down-sweep of the smoothing scan: the new trajectory (eq. 19) and the
// per-track largest change of the means.
template <class Model, typename R>
__global__ __launch_bounds__(kWave) void k_dn_backward_down(DnArgs a, int fan, const void* carry_in) {
  using D = Dense<Model, R>;
  constexpr int N = D::N;
  using Lay = typename D::Lay;
  __shared__ typename D::template WorkN<4> w;
  __shared__ R dmax[kWave];
  if (lane() == 0) w.ok = 1;
  const int64_t c = blockIdx.x;
  const int64_t s0 = c * fan;
  const int64_t s1 = min(s0 + fan, a.S);
  const int64_t nchunks = (a.S + fan - 1) / fan;
  R *cx = w.v[6], *cP = w.m[3];
  R *rE = w.m[0], *rL = w.m[1], *rg = w.v[0];
  bool have = c < nchunks - 1;
  if (have) D::load_carry(static_cast<const R*>(carry_in) + size_t(c) * Lay::kCarry, cx, cP);
  // running largest change of the current track segment of this chunk (lane 0);
  // published once per segment, and only when it exceeds the stored value
  int seg_track = -1;
  unsigned long long seg_bits = 0ull, all_bits = 0ull;
  auto publish = [&](unsigned long long* p, unsigned long long v) {
    if (v > *static_cast<volatile unsigned long long*>(p)) atomicMax(p, v);
  };
  for (int64_t k = 0; k < s1 - s0; ++k) {
    const int64_t s = s1 - 1 - k;
    D::load_selem(static_cast<const R*>(a.elem) + size_t(s) * Lay::kFElem, rE, rg, rL);
    if (have) {
      apply_s<N, R>(rE, rg, rL, cx, cP, w.m[2], w.v[2]);
    } else {
      vcopy<N>(rg, cx);
      copy<N, N, N, false>(rL, cP);
    }
    have = true;
    R* tj = static_cast<R*>(a.traj) + size_t(s) * Lay::kTraj;
    R m = R(0);
    bool nan = false;
    if (lane() < N) {
      const R d = fabs(cx[lane()] - tj[lane()]);
      nan = !(d == d);
      m = d;
    }
    dmax[lane()] = nan ? R(-1) : m;
    wsync();
    D::store_carry(cx, cP, tj);
    if (lane() == 0) {
      R mx = R(0);
      bool bad = false;
      for (int i = 0; i < N; ++i) {
        bad = bad || dmax[i] < R(0);
        mx = dmax[i] > mx ? dmax[i] : mx;
      }
      const unsigned long long bits = order_bits(bad ? __builtin_nan("") : double(mx));
      const int tr = a.track[s];
      if (tr != seg_track) {
        if (seg_track >= 0) publish(&a.delta_bits[seg_track], seg_bits);
        seg_track = tr;
        seg_bits = 0ull;
      }
      seg_bits = bits > seg_bits ? bits : seg_bits;
      all_bits = bits > all_bits ? bits : all_bits;
    }
    wsync();
  }
  if (lane() == 0 && seg_track >= 0) {
    publish(&a.delta_bits[seg_track], seg_bits);
    publish(&a.delta_bits[a.ntracks], all_bits);
  }
}

// Filtering pass only (Section 2: the filter is the prefix of the filtering
// elements): level 0 down-sweep that stores the filtered x*, P* of every slot
// of the chunk as a trajectory-layout record [slot][kTraj].
template <class Model, typename R>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(2))) void k_dn_forward_down_filter(DnArgs a, int fan, const void* carry_in,
                                                                  void* filt) {
  using D = Dense<Model, R>;
  constexpr int N = D::N;
  using Lay = typename D::Lay;
  __shared__ typename D::template WorkN<5> w;
  if (lane() == 0) w.ok = 1;
  const int64_t c = blockIdx.x;
  const int64_t s0 = c * fan;
  const int64_t s1 = min(s0 + fan, a.S);
  R *cx = w.v[6], *cP = w.m[4];
  R *rA = w.m[0], *rC = w.m[1], *rJ = w.m[2], *rb = w.v[0], *re = w.v[1];
  bool have = c > 0;
  if (have) D::load_carry(static_cast<const R*>(carry_in) + size_t(c) * Lay::kCarry, cx, cP);
  for (int64_t s = s0; s < s1; ++s) {
    D::load_felem(static_cast<const R*>(a.elem) + size_t(s) * Lay::kFElem, rA, rb, rC, re, rJ);
    if (have) {
      apply_f<N, R>(cx, cP, rA, rb, rC, re, rJ, w.m[3], w.v[2], w.v[3], &w.ok);
    } else {
      vcopy<N>(rb, cx);
      copy<N, N, N, false>(rC, cP);
    }
    have = true;
    D::store_carry(cx, cP, static_cast<R*>(filt) + size_t(s) * Lay::kTraj);
  }
}

// Log predictive density of slot s, log N(ytil_s; H_s m-_s + d_s, S_s) with
// m-_s = F x*_{s-1} + c, P-_s = F P*_{s-1} F^T + Q', S_s = H P-_s H^T + R'
// (the normalising constants that eq. 14 leaves out; summed over a track they
// give log p(y_{1:T}) of the linearised model), from the filtered moments of
// slot s-1; 0 at the first slot of a track.  One slot per workgroup.
template <class Model, typename R>
__global__ __launch_bounds__(kWave) void k_dn_loglik(DnArgs a, const void* filt, double* slot_ll) {
  using D = Dense<Model, R>;
  constexpr int N = D::N, P = D::P;
  using Lay = typename D::Lay;
  constexpr int L = ld<N>();
  __shared__ typename D::template WorkN<6> w;
  const int64_t s = blockIdx.x;
  if (a.flags[s] & kSlotFirst) {
    if (lane() == 0) slot_ll[s] = 0.0;
    return;
  }
  if (lane() == 0) w.ok = 1;
  const R* tr = static_cast<const R*>(a.trans) + size_t(s - 1) * Lay::kTrans;
  const R* hl = static_cast<const R*>(a.hlin) + size_t(s) * Lay::kHlin;
  const R* fp = static_cast<const R*>(filt) + size_t(s - 1) * Lay::kTraj;
  R *F = w.m[0], *Pf = w.m[1], *Pp = w.m[2], *HP = w.m[3], *H = w.m[4], *Sx = w.m[5];
  R *xf = w.v[0], *mp = w.v[1], *c = w.v[2], *d = w.v[3], *yt = w.v[4];
  ld_full<N, N, N>(tr, F);
  ld_v<N>(tr + N * N, c);
  ld_symm<N, N>(tr + N * N + N, Pp);
  ld_v<N>(fp, xf);
  ld_symm<N, N>(fp + N, Pf);
  ld_full<N, P, N>(hl, H);
  ld_v<P>(hl + P * N, d);
  ld_symm<N, P>(hl + P * N + P, Sx);
  ld_v<P>(hl + P * N + P + Lay::kSP, yt);
  wsync();
  mm<N, N, N, N, false, false>(F, Pf, (const R*)nullptr, R(1), HP);      // F P*
  mm<N, N, N, N, false, true>(HP, F, Pp, R(1), Pp);                      // P- = F P* F^T + Q'
  mv<N, N, N, false>(F, xf, c, R(1), mp);                                // m- = F x* + c
  mm<N, P, N, N, false, false>(H, Pp, (const R*)nullptr, R(1), HP);      // H P-
  mm<N, P, N, P, false, true>(HP, H, Sx, R(1), Sx);                      // S = H P- H^T + R'
  symmetrize<N, P>(Sx);
  chol<N, P>(Sx, &w.ok);
  mv<N, P, N, false>(H, mp, yt, R(-1), yt);                              // ytil - H m-
  for (int i = lane(); i < P; i += kWave) yt[i] -= d[i];
  wsync();
  fwd_vec<N, P>(Sx, yt);
  if (lane() == 0) {
    double quad = 0.0, logdet = 0.0;
    for (int i = 0; i < P; ++i) {
      quad += double(yt[i]) * double(yt[i]);
      logdet += 2.0 * log(double(Sx[i * L + i]));
    }
    constexpr double kLog2Pi = 1.8378770664093454836;
    slot_ll[s] = w.ok ? -0.5 * (P * kLog2Pi + logdet + quad) : __builtin_nan("");
  }
}

// Prior broadcast of the initial trajectory: (m0, P0) of the slot's track.
template <int N, typename R>
__global__ void k_dn_prior(int64_t S, const int* track, const R* m0, const R* P0, R* traj) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  constexpr int TW = N + sym_size<N>();
  if (e >= S * TW) return;
  const int64_t s = e / TW;
  const int k = int(e - s * TW);
  const int tr = track[s];
  if (k < N) {
    traj[e] = m0[size_t(tr) * N + k];
  } else {
    int i = 0, rem = k - N;
    while (rem >= N - i) {
      rem -= N - i;
      ++i;
    }
    traj[e] = P0[(size_t(tr) * N + i) * N + i + rem];
  }
}

// Caller layout <-> slot records: mean [S][N], cov [S][N][N].
template <int N, typename R>
__global__ void k_dn_unpack(int64_t S, const R* traj, R* mean, R* cov) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= S * N * N) return;
  const int64_t s = e / (N * N);
  const int r = int(e - s * N * N), i = r / N, j = r - i * N;
  const R* t = traj + size_t(s) * (N + sym_size<N>());
  if (cov) cov[e] = t[N + sym_index<N>(i, j)];
  if (mean && j == 0) mean[s * N + i] = t[i];
}

template <int N, typename R>
__global__ void k_dn_pack(int64_t S, const R* mean, const R* cov, SymConst<N, R> cc, int use_const, const int* track,
                          const R* P0, R* traj) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  constexpr int TW = N + sym_size<N>();
  if (e >= S * TW) return;
  const int64_t s = e / TW;
  const int k = int(e - s * TW);
  if (k < N) {
    traj[e] = mean[s * N + k];
    return;
  }
  int i = 0, rem = k - N;
  while (rem >= N - i) {
    rem -= N - i;
    ++i;
  }
  const int j = i + rem;
  if (cov)
    traj[e] = R(0.5) * (cov[(s * N + i) * N + j] + cov[(s * N + j) * N + i]);
  else if (use_const)
    traj[e] = cc.v[k - N];
  else
    traj[e] = P0[(size_t(track[s]) * N + i) * N + j];
}

}  // namespace dn
}  // namespace pks
