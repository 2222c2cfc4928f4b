// Kernels of the warm-start network: a patch-embedding 1-D convolution,
// dilated residual convolutions and a per-patch linear head, FP32, with the
// backward pass and Adam.  Activations are channel-major, [channels][n * L]
// (window-major positions inside a channel row), so every convolution is a
// GEMM whose right operand is gathered on the fly from the source rows.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "wgrad_chunks.hpp"

namespace wsn {

constexpr int kThreads = 256; // 16 x 16 threads, 4 x 4 outputs each
constexpr int kPad = 4;       // LDS row padding: column writes of 16 rows hit distinct banks

// B(r, p) of a convolution: r = c * K + k (source row c, tap k), p = w * Lout + j
// (window w, output position j); the source position is j * stride + k * dil - pad,
// zero outside [0, Lin).
struct Gather {
  const float* src;  // [rows][ld]
  int ld;            // n * Lin
  int K, Lout, Lin, stride, dil, pad;
};

__device__ __forceinline__ float gather_at(const Gather& g, int r, int p) {
  const int c = r / g.K, k = r - c * g.K;
  const int w = p / g.Lout, j = p - w * g.Lout;
  const int s = j * g.stride + k * g.dil - g.pad;
  return (s >= 0 && s < g.Lin) ? g.src[size_t(c) * g.ld + size_t(w) * g.Lin + s] : 0.f;
}

enum Epilogue { kEpiRelu = 0, kEpiResidual = 1, kEpiLinear = 2, kEpiBackward = 3 };

struct ConvArgs {
  int M, Kr, N;          // output rows, reduction length, output positions (N % 4 == 0)
  const float* W;        // weights [Cout][Cin][K]
  int transposed;        // 0: A(m, r) = W[m * Kr + r]; 1: A(m, r = co * K + k) = W[(co * M + m) * K + k]
  const float* bias;     // [M] (forward epilogues)
  Gather g;
  float* out;            // relu: h; residual: relu part a; linear: output; backward: dh (nullable)
  float* out2;           // residual: h_prev + a; backward: dh masked by (mask > 0)
  const float* in2;      // residual: h_prev; backward: dh of the layer above (nullable)
  const float* mask;     // backward: relu output of the source layer
};

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void st4(float* p, float4 v) { *reinterpret_cast<float4*>(p) = v; }

// One reduction stage of a 64 x 64 output tile: As[rr][mm] = A(m0 + mm, r0 + rr),
// Bs[rb][pp] = B(r0 + rb, p0 + pp), zero outside the matrices.
__device__ __forceinline__ void stage_tile(const ConvArgs& a, int t, int m0, int p0, int r0,
                                           float (&As)[kTk][kTile + kPad], float (&Bs)[kTk][kTile]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = t + kThreads * i;
    // weights: consecutive lanes take consecutive addresses of W in both forms
    if (a.transposed) {
      const int mm = e & 63, rr = e >> 6, m = m0 + mm, r = r0 + rr;
      float v = 0.f;
      if (m < a.M && r < a.Kr) {
        const int co = r / a.g.K, k = r - co * a.g.K;
        v = a.W[(size_t(co) * a.M + m) * a.g.K + k];
      }
      As[rr][mm] = v;
    } else {
      const int rr = e & 15, mm = e >> 4, m = m0 + mm, r = r0 + rr;
      As[rr][mm] = (m < a.M && r < a.Kr) ? a.W[size_t(m) * a.Kr + r] : 0.f;
    }
    const int pp = e & 63, rb = e >> 6, p = p0 + pp, r = r0 + rb;
    Bs[rb][pp] = (p < a.N && r < a.Kr) ? gather_at(a.g, r, p) : 0.f;
  }
}

// out[m][p] = epilogue(sum_r A(m, r) B(r, p)), residual or backward: the layers
// whose windows do not fill the tiles of k_conv_direct.  grid (ceil(N / 64),
// ceil(M / 64)).
template <int EPI>
__global__ __launch_bounds__(kThreads) void k_conv(ConvArgs a) {
  static_assert(EPI == kEpiResidual || EPI == kEpiBackward, "the other layers run k_conv_direct");
  __shared__ __align__(16) float As[kTk][kTile + kPad];
  __shared__ __align__(16) float Bs[kTk][kTile];
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
  const int m0 = blockIdx.y * kTile, p0 = blockIdx.x * kTile;
  float acc[4][4] = {};
  for (int r0 = 0; r0 < a.Kr; r0 += kTk) {
    stage_tile(a, t, m0, p0, r0, As, Bs);
    __syncthreads();
#pragma unroll
    for (int rr = 0; rr < kTk; ++rr) {
      const float4 av = ld4(&As[rr][4 * ty]);
      const float4 bv = ld4(&Bs[rr][4 * tx]);
      const float ar[4] = {av.x, av.y, av.z, av.w};
      const float br[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(ar[i], br[j], acc[i][j]);
    }
    __syncthreads();
  }
  const int p = p0 + 4 * tx;
  if (p >= a.N) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + 4 * ty + i;
    if (m >= a.M) break;
    const size_t o = size_t(m) * a.N + p;
    float4 v = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    if (EPI == kEpiBackward) {
      if (a.in2) {
        const float4 u = ld4(a.in2 + o);
        v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
      }
      if (a.out) st4(a.out + o, v);
      const float4 mk = ld4(a.mask + o);
      st4(a.out2 + o, make_float4(mk.x > 0.f ? v.x : 0.f, mk.y > 0.f ? v.y : 0.f,
                                  mk.z > 0.f ? v.z : 0.f, mk.w > 0.f ? v.w : 0.f));
    } else {
      const float b = a.bias[m];
      v.x += b; v.y += b; v.z += b; v.w += b;
      v = make_float4(fmaxf(v.x, 0.f), fmaxf(v.y, 0.f), fmaxf(v.z, 0.f), fmaxf(v.w, 0.f));
      st4(a.out + o, v);
      const float4 u = ld4(a.in2 + o);
      st4(a.out2 + o, make_float4(u.x + v.x, u.y + v.y, u.z + v.z, u.w + v.w));
    }
  }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// The same convolutions on the FP32 matrix cores, for layers whose output
// positions are their source's (the residual layers, with KT = 3 taps, when
// whole windows fill tiles of 64 positions; embedding and head, KT = 1).  A
// block takes 32 PW positions and 128 output rows; up to 128 source channels
// go through LDS as they lie in memory, so that a tap is a shifted LDS read,
// masked at the window's edges, and no index is divided per element (the
// gather of k_conv cost more than its multiply-adds).  The weights are packed
// in the order in which the lanes take them (k_pack) and come straight
// from the caches: through LDS they took the registers of a second block per CU.
// 128 x 384 x 16,384: 77 us with k_conv, 30 to 34 here; bound by the
// products (10 us at the card's FP32 matrix rate) and 33 MB of activations.
// 16 x 16 x 4 FP32 MFMA: lane l feeds A[l % 16][l / 16] and B[l / 16][l % 16],
// four channels of one tap per instruction, and receives D[4 (l / 16) + q][l %
// 16].  It adds its four products one after the other, each rounded as a
// multiply-add, and they are taken in the order of the reduction index (channel,
// tap), so the sums are k_conv's bit for bit, at twice the vector unit's rate.
// Each wave owns 32 x 32 (waves without rows only stage).  grid (ceil(N / (32
// PW)), ceil(M / 128)), 256 PW threads.
// ---------------------------------------------------------------------------
struct DirectArgs {
  int M, Cin, N, Lpos;   // output rows, source channels, positions, positions per window
  const float* W;        // packed weights (PackDirect)
  const float* bias;     // [M] (forward epilogues)
  const float* src;      // channel c at position p: src[(c / patch) ld + p patch + c % patch]
  int ld, patch;
  int dil;               // tap k reads position p + (k - 1) dil of the same window
  float* out;            // as in ConvArgs
  float* out2;
  const float* in2;
  const float* mask;
};

// A layer's weights as A fragments: word ((mt S + s) 64 + l) 4 + e, S = KT ceil(
// Cin / 16), s = (group of 16 channels) KT + f: row 16 mt + l % 16, reduction
// index r = 4 (4 f + e) + l / 16 of the group, channel 16 group + r / KT, tap
// r % KT, zero past the matrix.  Row tiles are padded to pairs.
struct PackDirect {
  const float* W;        // [Cout][Cin][K] of the layer
  int M, Cin, KT;        // rows and channels as the convolution sees them
  int transposed;        // 0: A(m, c, k) = W[(m Cin + c) K + k]; 1: W[(c M + m) K + k]
  float* out;
};
__host__ __device__ __forceinline__ int64_t direct_words(int M, int Cin, int KT) {
  return int64_t((M + 31) / 32) * 2 * KT * ((Cin + 15) / 16) * 256;
}
__device__ __forceinline__ void pack_direct(const PackDirect& a) {
  const int64_t words = direct_words(a.M, a.Cin, a.KT);
  const int S = a.KT * ((a.Cin + 15) / 16);
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < words; i += int64_t(gridDim.x) * 256) {
    const int e = int(i & 3), l = int(i >> 2) & 63;
    const int64_t t = i >> 8;
    const int s = int(t % S), r = 4 * (4 * (s % a.KT) + e) + (l >> 4);
    const int m = int(t / S) * 16 + (l & 15), c = 16 * (s / a.KT) + r / a.KT, k = r % a.KT;
    float v = 0.f;
    if (m < a.M && c < a.Cin)
      v = a.W[(a.transposed ? int64_t(c) * a.M + m : int64_t(m) * a.Cin + c) * a.KT + k];
    a.out[i] = v;
  }
}

constexpr int kDirC = 128;   // source channels per stage

template <int KT, int EPI, int PW>
__global__ __launch_bounds__(256 * PW) void k_conv_direct(DirectArgs a) {
  constexpr int T = 256 * PW, P = 32 * PW;
  constexpr int BP = P + 16;     // row pitch: the four channel rows of a fragment on distinct banks
  __shared__ float Bs[kDirC][BP];
  const int t = threadIdx.x, wv = t >> 6, ln = t & 63, g = ln >> 4, lr = ln & 15;
  const int p0 = blockIdx.x * P;
  const int m0 = (blockIdx.y * 4 + wv / PW) * 32, pw = (wv % PW) * 32;   // this wave's part of the output
  // Step u of a channel group takes r = 4 u + g, i.e. channel (4 u + g) / KT and
  // tap (4 u + g) % KT: of the three cases v = u % 3 (KT = 3), this lane's LDS
  // row past 4 u / 3, its column in each position tile, and whether that lies
  // in the window.
  int at[KT][2];
  bool live[KT][2];
#pragma unroll
  for (int v = 0; v < KT; ++v)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int row = KT == 3 ? (v + g) / 3 : g, k = KT == 3 ? (v + g) % 3 : 0;
      const int p = pw + 16 * j + lr, off = KT == 3 ? (k - 1) * a.dil : 0;
      const int q = KT == 3 ? p % a.Lpos + off : 0;
      live[v][j] = KT == 1 || (q >= 0 && q < a.Lpos);
      at[v][j] = row * BP + (live[v][j] ? p + off : p);
    }
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int S = KT * ((a.Cin + 15) / 16);
  const bool rows = m0 < a.M;
  const f32x4* W = reinterpret_cast<const f32x4*>(a.W) + (int64_t(rows ? m0 : 0) / 16 * S) * 64 + ln;
  for (int c0 = 0; c0 < a.Cin; c0 += kDirC) {
    const int cn = min(kDirC, (a.Cin - c0 + 15) & ~15);   // channels of this stage, padded to whole groups
    if (c0 > 0) __syncthreads();
#pragma unroll 8
    for (int e = t; e < cn * P; e += T) {
      const int c = c0 + e / P, p = p0 + e % P;
      const int row = a.patch == 1 ? c : c / a.patch;
      Bs[e / P][e % P] =
          (c < a.Cin && p < a.N) ? a.src[size_t(row) * a.ld + size_t(p) * a.patch + (c - row * a.patch)] : 0.f;
    }
    __syncthreads();
    const f32x4* w = W + int64_t(c0 / 16) * KT * 64;
    for (int cg = 0; rows && cg < cn / 16; ++cg)
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        f32x4 x[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) x[i] = w[(int64_t(i) * S + cg * KT + k) * 64];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int u = 4 * k + e, v = KT == 3 ? u % 3 : 0;
          float y[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float b = Bs[16 * cg + 4 * u / KT][at[v][j]];
            y[j] = live[v][j] ? b : 0.f;
          }
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][e], y[j], acc[i][j], 0, 0, 0);
        }
      }
  }
  if (!rows) return;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = m0 + 16 * i + 4 * g + q;
      if (m >= a.M) continue;
      const float b = EPI == kEpiBackward ? 0.f : a.bias[m];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int p = p0 + pw + 16 * j + lr;
        if (p >= a.N) continue;
        const size_t o = size_t(m) * a.N + p;
        float v = acc[i][j][q];
        if (EPI == kEpiBackward) {
          if (a.in2) v += a.in2[o];
          if (a.out) a.out[o] = v;
          a.out2[o] = a.mask[o] > 0.f ? v : 0.f;
        } else if (EPI == kEpiLinear) {
          a.out[o] = v + b;
        } else {
          v = fmaxf(v + b, 0.f);
          a.out[o] = v;
          if (EPI == kEpiResidual) a.out2[o] = a.in2[o] + v;
        }
      }
    }
}

// ---------------------------------------------------------------------------
// Inference form of the forward convolutions on the matrix cores: the same
// tiles and staging as k_conv, the products as 16 x 16 x 16 BF16 MFMA with
// FP32 accumulation (operands rounded to BF16, to nearest even).  Each of the
// four waves owns a 32 x 32 quarter of the 64 x 64 tile, two by two MFMA
// blocks.  Operand layout of the MFMA (lane l, element j): A[l % 16][4 (l / 16)
// + j], B[4 (l / 16) + j][l % 16]; result D[4 (l / 16) + j][l % 16].
// Forward epilogues only (bias + ReLU, residual, linear).
// ---------------------------------------------------------------------------
typedef short bf16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return short(u >> 16);
}

template <int EPI>
__global__ __launch_bounds__(kThreads) void k_conv_mfma(ConvArgs a) {
  static_assert(EPI != kEpiBackward, "forward epilogues only");
  __shared__ __align__(16) float As[kTk][kTile + kPad];
  __shared__ __align__(16) float Bs[kTk][kTile];
  const int t = threadIdx.x, wv = t >> 6, ln = t & 63;
  const int m0 = blockIdx.y * kTile, p0 = blockIdx.x * kTile;
  const int mw = (wv >> 1) * 32, nw = (wv & 1) * 32;   // this wave's quarter of the tile
  const int kq = 4 * (ln >> 4), lr = ln & 15;
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int r0 = 0; r0 < a.Kr; r0 += kTk) {
    stage_tile(a, t, m0, p0, r0, As, Bs);
    __syncthreads();
    bf16x4 af[2], bf[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        af[i][j] = to_bf16(As[kq + j][mw + 16 * i + lr]);
        bf[i][j] = to_bf16(Bs[kq + j][nw + 16 * i + lr]);
      }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(af[i], bf[j], acc[i][j], 0, 0, 0);
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + mw + 16 * i + kq + q, p = p0 + nw + 16 * j + lr;
        if (m >= a.M || p >= a.N) continue;
        const size_t o = size_t(m) * a.N + p;
        float v = acc[i][j][q] + a.bias[m];
        if (EPI == kEpiLinear) {
          a.out[o] = v;
        } else {
          v = fmaxf(v, 0.f);
          a.out[o] = v;
          if (EPI == kEpiResidual) a.out2[o] = a.in2[o] + v;
        }
      }
}

// Weight gradient partials: part[z][m][r] = sum over the z-th chunk of
// positions of D[m][p] B(r, p), with r = Kr the bias column (B = 1).
// grid (ceil((Kr + 1) / 64), ceil(M / 64), chunks).
struct WgradArgs {
  int M, Kr, N, chunk;
  const float* D;   // [M][N]
  Gather g;
  float* part;      // [chunks][M][Kr + 1]
};

__global__ __launch_bounds__(kThreads) void k_wgrad(WgradArgs a) {
  __shared__ __align__(16) float Ds[kTk][kTile + kPad];
  __shared__ __align__(16) float Bs[kTk][kTile + kPad];
  const int t = threadIdx.x, tx = t & 15, ty = t >> 4;
  const int r0 = blockIdx.x * kTile, m0 = blockIdx.y * kTile;
  const int pbeg = blockIdx.z * a.chunk;
  const int pend = min(pbeg + a.chunk, a.N);
  const int R1 = a.Kr + 1;
  float acc[4][4] = {};
  for (int pc = pbeg; pc < pend; pc += kTk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = t + kThreads * i, pp = e & 15, q = e >> 4;   // q: row (m or r) within the tile
      const int p = pc + pp;
      const bool live = p < pend;
      const int m = m0 + q;
      Ds[pp][q] = (live && m < a.M) ? a.D[size_t(m) * a.N + p] : 0.f;
      const int r = r0 + q;
      float bv = 0.f;
      if (live && r < R1) bv = r == a.Kr ? 1.f : gather_at(a.g, r, p);
      Bs[pp][q] = bv;
    }
    __syncthreads();
#pragma unroll
    for (int pp = 0; pp < kTk; ++pp) {
      const float4 dv = ld4(&Ds[pp][4 * ty]);
      const float4 bv = ld4(&Bs[pp][4 * tx]);
      const float dr[4] = {dv.x, dv.y, dv.z, dv.w};
      const float br[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(dr[i], br[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + 4 * ty + i;
    if (m >= a.M) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + 4 * tx + j;
      if (r < R1) a.part[(size_t(blockIdx.z) * a.M + m) * R1 + r] = acc[i][j];
    }
  }
}

// Weight-gradient partials of the same layers on the FP32 matrix cores: the
// positions are the reduction, so a lane's A is D[m][p] and its B the source
// channel at p + (k - 1) dil, four positions per instruction; a block takes
// 128 rows, 32 channels with all their taps, and `chunk` positions (a multiple
// of 64), in stages of 64.  Against k_wgrad, whose gather ran once per element
// and tile: 128 x 385 over 16,384 positions 75 us, 30 here.
// grid (ceil(Cin / 32), ceil(M / 128), chunks).
struct DirectWgradArgs {
  int M, Cin, N, Lpos, chunk;
  const float* D;        // [M][N]
  const float* src;      // as in DirectArgs
  int ld, patch, dil;
  float* part;           // [chunks][M][Cin KT + 1]
};

template <int KT>
__global__ __launch_bounds__(256) void k_wgrad_direct(DirectWgradArgs a) {
  constexpr int T = 256, MR = 128, CR = 32;
  constexpr int PP = kDirP + 4;     // row pitch: the 16 rows x 4 positions of a fragment on distinct banks
  __shared__ float Ds[MR][PP];
  __shared__ float Bs[CR][PP];
  const int t = threadIdx.x, wv = t >> 6, ln = t & 63, g = ln >> 4, lr = ln & 15;
  const int m0 = blockIdx.y * MR, cb = blockIdx.x * CR;
  const int pbeg = blockIdx.z * a.chunk, pend = min(pbeg + a.chunk, a.N);
  f32x4 acc[2][2][KT];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < KT; ++k) acc[i][j][k] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bias[2] = {0.f, 0.f};
  constexpr int DN = MR * kDirP / T, BN = CR * kDirP / T;
  float dv[DN], bv[BN];
  auto load = [&](int pc) {
#pragma unroll
    for (int i = 0; i < DN; ++i) {
      const int e = t + T * i, m = m0 + e / kDirP, p = pc + e % kDirP;
      dv[i] = (m < a.M && p < pend) ? a.D[size_t(m) * a.N + p] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < BN; ++i) {
      const int e = t + T * i, c = cb + e / kDirP, p = pc + e % kDirP;
      const int row = a.patch == 1 ? c : c / a.patch;
      bv[i] = (c < a.Cin && p < pend) ? a.src[size_t(row) * a.ld + size_t(p) * a.patch + (c - row * a.patch)] : 0.f;
    }
  };
  load(pbeg);
  for (int pc = pbeg; pc < pend; pc += kDirP) {
#pragma unroll
    for (int i = 0; i < DN; ++i) Ds[(t + T * i) / kDirP][(t + T * i) % kDirP] = dv[i];
#pragma unroll
    for (int i = 0; i < BN; ++i) Bs[(t + T * i) / kDirP][(t + T * i) % kDirP] = bv[i];
    __syncthreads();
    if (pc + kDirP < pend) load(pc + kDirP);
#pragma unroll 4
    for (int s = 0; m0 + 32 * wv < a.M && s < kDirP / 4; ++s) {
      const int p = 4 * s + g;
      float x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        x[i] = Ds[32 * wv + 16 * i + lr][p];
        bias[i] += x[i];
      }
      const int w = KT == 3 ? p % a.Lpos : 0;
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        const int off = KT == 3 ? (k - 1) * a.dil : 0;
        const bool live = KT == 1 || (w + off >= 0 && w + off < a.Lpos);
        const int q = live ? p + off : p;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const float v = Bs[16 * j + lr][q];
          const float y = live ? v : 0.f;
#pragma unroll
          for (int i = 0; i < 2; ++i) acc[i][j][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y, acc[i][j][k], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  const int Kr = a.Cin * KT;
  float* part = a.part + size_t(blockIdx.z) * a.M * (Kr + 1);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = m0 + 32 * wv + 16 * i + 4 * g + q;
      if (m >= a.M) continue;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = cb + 16 * j + lr;
        if (c >= a.Cin) continue;
#pragma unroll
        for (int k = 0; k < KT; ++k) part[size_t(m) * (Kr + 1) + c * KT + k] = acc[i][j][k][q];
      }
    }
    // bias column: the sums of D over this lane's quarter of the positions
    float b = bias[i];
    b += __shfl_xor(b, 16);
    b += __shfl_xor(b, 32);
    const int m = m0 + 32 * wv + 16 * i + lr;
    if (blockIdx.x == 0 && g == 0 && m < a.M) part[size_t(m) * (Kr + 1) + Kr] = b;
  }
}

// Sums the chunk partials into the flat gradient: W part at w_off + m * Kr + r,
// bias at b_off + m.  A block takes 64 entries; its four waves sum a quarter of
// the chunks each, in order, and the quarters are added in order.  (One thread
// per entry over all chunks left 193 blocks waiting on 64 loads in a row: 25 us
// for 128 x 385 over 64 chunks, 5 us now.)
__global__ __launch_bounds__(256) void k_wgrad_reduce(const float* part, int chunks, int M, int Kr, float* grad,
                                                      int64_t w_off, int64_t b_off) {
  __shared__ float sum[4][64];
  const int R1 = Kr + 1, ln = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t e = int64_t(blockIdx.x) * 64 + ln, cnt = int64_t(M) * R1;
  const int z0 = chunks * wv / 4, z1 = chunks * (wv + 1) / 4;
  float s = 0.f;
  if (e < cnt) {
#pragma unroll 8
    for (int z = z0; z < z1; ++z) s += part[z * cnt + e];
  }
  sum[wv][ln] = s;
  __syncthreads();
  if (wv > 0 || e >= cnt) return;
  s = ((sum[0][ln] + sum[1][ln]) + sum[2][ln]) + sum[3][ln];
  const int64_t m = e / R1, r = e - m * R1;
  if (r < Kr) grad[w_off + m * Kr + r] = s;
  else grad[b_off + m] = s;
}

// Mean-squared error: dout = scale * (out - target), scale = 2 / count; block
// partial sums of the squared error (fixed order) into part[blockIdx.x].
__global__ __launch_bounds__(256) void k_mse(const float* out, const float* target, float* dout, int64_t count,
                                             float scale, float* part) {
  __shared__ float red[256];
  float s = 0.f;
  for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < count; e += int64_t(gridDim.x) * 256) {
    const float d = out[e] - target[e];
    dout[e] = scale * d;
    s = fmaf(d, d, s);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_sum(const float* part, int n, float scale, float* out) {
  __shared__ float red[256];
  float s = 0.f;
  for (int e = threadIdx.x; e < n; e += 256) s += part[e];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = red[0] * scale;
}

// Adam (Kingma & Ba, 2015) with bias corrections c1 = 1 - beta1^t, c2 = 1 - beta2^t.
__global__ void k_adam(float* theta, const float* g, float* m, float* v, int64_t n, float lr, float beta1,
                       float beta2, float eps, float c1, float c2) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const float gi = g[e];
  const float mi = beta1 * m[e] + (1.f - beta1) * gi;
  const float vi = beta2 * v[e] + (1.f - beta2) * gi * gi;
  m[e] = mi;
  v[e] = vi;
  theta[e] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Windows of the planned tracks (device tables).
struct WindowTable {
  const int* track;        // [n_windows] track of each window
  const int* start;        // [n_windows] first step (1-based) of each window
  const int64_t* meas_off; // [n_tracks + 1] measurement offsets
  const int* first;        // [n_tracks + 1] first window of each track
};

// Network inputs of windows w0 .. w0 + n - 1: (sin, cos) of every bearing.
// channel_major: x[c][b * W + t] (a batch), else x[b][c][t] (a data set).
__global__ void k_features(WindowTable tab, const double* y, int ny, int W, int64_t w0, int n, int channel_major,
                           float* x) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= int64_t(n) * W) return;
  const int b = int(e / W), t = int(e - int64_t(b) * W);
  const int64_t w = w0 + b;
  const int tr = tab.track[w];
  const int64_t T = tab.meas_off[tr + 1] - tab.meas_off[tr];
  const int64_t k = min(int64_t(tab.start[w]) + t, T);
  const double* yk = y + (tab.meas_off[tr] + k - 1) * ny;
  const int cin = 2 * ny;
  for (int s = 0; s < ny; ++s) {
    double sv, cv;
    sincos(yk[s], &sv, &cv);
    const size_t i0 = channel_major ? size_t(2 * s) * n * W + size_t(b) * W + t : (size_t(b) * cin + 2 * s) * W + t;
    const size_t i1 = channel_major ? i0 + size_t(n) * W : i0 + W;
    x[i0] = float(sv);
    x[i1] = float(cv);
  }
}

// Labels of every window from smoothed means [S][nx]: lab[w][t][i].
__global__ void k_labels(WindowTable tab, const double* mean, int nx, int W, int64_t n_windows, float* lab) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= n_windows * W) return;
  const int64_t w = e / W;
  const int t = int(e - w * W);
  const int tr = tab.track[w];
  const int64_t T = tab.meas_off[tr + 1] - tab.meas_off[tr];
  const int64_t k = min(int64_t(tab.start[w]) + t, T);
  const int64_t slot = tab.meas_off[tr] + tr + k;
  for (int i = 0; i < nx; ++i) lab[e * nx + i] = float(mean[slot * nx + i]);
}

// Batch assembly from a data set of n_data windows: xb[c][b * W + t] =
// x[idx[b]][c][t]; when lab is given, tb[u * nx + i][b * L + j] =
// (lab[idx[b]][P j + u][i] - mu_i) / sigma_i.  An index outside [0, n_data)
// reads nothing: its window is zero and *bad is set.
__global__ void k_gather_batch(const float* x, const float* lab, int64_t n_data, const int* idx, int n, int cin,
                               int W, int P, int nx, const float* mu, const float* sigma, float* xb, float* tb,
                               int* bad) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= int64_t(n) * W) return;
  const int b = int(e / W), t = int(e - int64_t(b) * W);
  const int64_t src = idx[b];
  const bool ok = src >= 0 && src < n_data;
  if (!ok && t == 0) atomicOr(bad, 1);
  for (int c = 0; c < cin; ++c) xb[size_t(c) * n * W + e] = ok ? x[(src * cin + c) * W + t] : 0.f;
  if (lab) {
    const int L = W / P, j = t / P, u = t - j * P;
    for (int i = 0; i < nx; ++i)
      tb[size_t(u * nx + i) * n * L + size_t(b) * L + j] =
          ok ? (lab[(src * W + t) * nx + i] - mu[i]) / sigma[i] : 0.f;
  }
}

// Network outputs [P nx][n L] -> states out[b][t][i] = mu_i + sigma_i * o.
__global__ void k_states(const float* o, int n, int W, int P, int nx, const float* mu, const float* sigma,
                         float* out) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= int64_t(n) * W) return;
  const int b = int(e / W), t = int(e - int64_t(b) * W);
  const int L = W / P, j = t / P, u = t - j * P;
  for (int i = 0; i < nx; ++i)
    out[e * nx + i] = mu[i] + sigma[i] * o[size_t(u * nx + i) * n * L + size_t(b) * L + j];
}

// Network outputs of windows w0 .. w0 + n - 1 -> initial trajectory mean[S][nx]
// (FP64): step k of a track comes from window min((k - 1) / W, n_w - 1) of that
// track, slot 0 from step 1.
__global__ void k_scatter(WindowTable tab, const float* o, int64_t w0, int n, int W, int P, int nx,
                          const float* mu, const float* sigma, double* mean) {
  const int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (e >= int64_t(n) * W) return;
  const int b = int(e / W), t = int(e - int64_t(b) * W);
  const int64_t w = w0 + b;
  const int tr = tab.track[w];
  const int64_t T = tab.meas_off[tr + 1] - tab.meas_off[tr];
  const int64_t k = int64_t(tab.start[w]) + t;
  if (k > T) return;
  const int nw = tab.first[tr + 1] - tab.first[tr];
  const int64_t owner = tab.first[tr] + min((k - 1) / W, int64_t(nw - 1));
  if (owner != w) return;
  const int L = W / P, j = t / P, u = t - j * P;
  const int64_t slot = tab.meas_off[tr] + tr + k;
  for (int i = 0; i < nx; ++i) {
    const double v = double(mu[i] + sigma[i] * o[size_t(u * nx + i) * n * L + size_t(b) * L + j]);
    mean[slot * nx + i] = v;
    if (k == 1) mean[(slot - 1) * nx + i] = v;
  }
}

// ---------------------------------------------------------------------------
// Inference form of the whole network on the matrix cores (width C = 128 or
// 256, whole windows in a tile of 128 positions): features, embedding, every
// residual layer, head, and the scatter into the trajectory, in one kernel.
// Windows do not interact, so a block takes kNetP positions (whole windows)
// through all layers: the FP32 residual stream stays in registers, in the
// MFMA result layout that the next layer's epilogue needs again, and only its
// BF16 rounding goes through LDS, position-major, as the next layer's B
// operand.  HBM sees the measurements and the trajectory alone; one kernel per
// layer moved the stream through HBM twice per layer (C = 128, four residual
// layers, 32,768 windows of 16 positions: 1.39 ms a call, 0.35 now).
// Bound: the BF16 products (206 GFLOP), their LDS reads (each wave reads the
// whole tile for its C / 4 rows) close behind.
//
// Products are 16 x 16 x 16 BF16 MFMA with FP32 accumulation, reduction in
// order of (tap, channel): operands of k_conv_mfma, element for element.  Two
// of its 16-deep steps are stored side by side -- channel 16 h + 4 g + j of a
// group of 32 sits at 8 g + 4 h + j (net_col) -- so that one 16-byte read
// feeds both, of the LDS tile and of the weights, which are packed in the
// order in which the lanes take them (k_pack).
// ---------------------------------------------------------------------------
constexpr int kNetP = 128;   // positions per block
typedef short bf16x8 __attribute__((ext_vector_type(8)));

__host__ __device__ __forceinline__ int net_col(int c) {
  return (c & ~31) | ((c & 12) << 1) | ((c & 16) >> 2) | (c & 3);
}

// 16-row tiles and 32-deep steps of a packed weight matrix of M rows and Kr columns.
__host__ __device__ __forceinline__ int net_steps(int Kr) { return (Kr + 31) / 32; }
__host__ __device__ __forceinline__ int64_t net_words(int M, int Kr) {
  return int64_t((M + 15) / 16) * net_steps(Kr) * 512;
}

// A weight matrix [M][cin][K] as BF16 fragments: word 8 l + e of (row tile mt,
// step s) is row 16 mt + l % 16, reduction index r = 32 s + 16 (e / 4) +
// 4 (l / 16) + e % 4, zero past the matrix.  Reduction order: taps outermost
// when tap_major (r = k cin + c), else r = c K + k.
struct PackNet {
  const float* W;
  int M, cin, K, tap_major;
  short* out;
};
__device__ __forceinline__ void pack_net(const PackNet& a) {
  const int Kr = a.cin * a.K, steps = net_steps(Kr);
  const int64_t words = net_words(a.M, Kr);
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < words; i += int64_t(gridDim.x) * 256) {
    const int e = int(i & 7), l = int(i >> 3) & 63;
    const int64_t t = i >> 9;
    const int s = int(t % steps), m = int(t / steps) * 16 + (l & 15);
    const int r = 32 * s + 16 * (e >> 2) + 4 * (l >> 4) + (e & 3);
    float v = 0.f;
    if (m < a.M && r < Kr) {
      const int c = a.tap_major ? r % a.cin : r / a.K, k = a.tap_major ? r / a.cin : r - c * a.K;
      v = a.W[(int64_t(m) * a.cin + c) * a.K + k];
    }
    a.out[i] = to_bf16(v);
  }
}

// Every packed copy of the weights in one launch, grid (blocks, n_direct + n_net).
constexpr int kPackDirect = 32, kPackNet = 16;
struct PackArgs {
  PackDirect direct[kPackDirect];
  PackNet net[kPackNet];
  int n_direct, n_net;
};
__global__ __launch_bounds__(256) void k_pack(PackArgs a) {
  const int i = blockIdx.y;
  if (i < a.n_direct) pack_direct(a.direct[i]);
  else pack_net(a.net[i - a.n_direct]);
}

struct NetArgs {
  WindowTable tab;
  const double* y;
  double* mean;
  int64_t w0, n;                 // first window, windows of this launch
  int ny, W, P, nx, Lpos, hidden;
  const short *we, *wr, *wh;     // packed embedding, residual layers, head
  const float *be, *bh;          // biases of the embedding and the head
  const float* br;               // bias of the first residual layer; the next one's br_stride later
  int64_t br_stride;
  const float *mu, *sigma;
  const float* h0;               // !kEmbed: output of the embedding [C][n Lpos]
  float* h1;                     // !kHead: takes the output of the last residual layer
};

// Without kEmbed the embedding's output is read, without kHead the last layer's
// is written (variants: with both forms in one kernel its registers spill, 422 us
// instead of 375 for 32,768 windows).
template <int C, bool kEmbed, bool kHead>
__global__ __launch_bounds__(256, C == 128 ? 2 : 1) void k_net_mfma(NetArgs a) {
  static_assert(C % 128 == 0, "whole 32-row pairs of tiles per wave");
  constexpr int RT = C / 64;     // 16-row tiles per wave
  constexpr int NT = kNetP / 16;  // 16-position tiles
  constexpr int CP = C + 8;      // LDS row pitch (BF16): rows 16 B apart in bank order
  __shared__ __align__(16) short Hs[kNetP + 1][CP];   // last row: zeros, for taps outside the window
  const int t = threadIdx.x, wv = t >> 6, ln = t & 63, g = ln >> 4, lr = ln & 15;
  const int64_t p0 = int64_t(blockIdx.x) * kNetP;     // of this launch's positions
  const int64_t N = a.n * a.Lpos;
  for (int c = t; c < CP; c += 256) Hs[kNetP][c] = 0;

  f32x4 h[RT][NT], acc[RT][NT];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // acc += W[rows of this wave][steps s0 ..] x Hs[row[j]], columns 0 .. 32 n
  auto product = [&](const short* w, int steps, int s0, int n, const int (&row)[NT]) {
    const short* wp = w + (int64_t(wv * RT) * steps + s0) * 512 + ln * 8;
#pragma unroll 2
    for (int s = 0; s < n; ++s) {
      bf16x8 af[RT];
#pragma unroll
      for (int i = 0; i < RT; ++i) af[i] = *reinterpret_cast<const bf16x8*>(wp + (int64_t(i) * steps + s) * 512);
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(&Hs[row[j]][32 * s + 8 * g]);
        const bf16x4 b0 = __builtin_shufflevector(b, b, 0, 1, 2, 3), b1 = __builtin_shufflevector(b, b, 4, 5, 6, 7);
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const bf16x4 a0 = __builtin_shufflevector(af[i], af[i], 0, 1, 2, 3);
          const bf16x4 a1 = __builtin_shufflevector(af[i], af[i], 4, 5, 6, 7);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, b0, acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, b1, acc[i][j], 0, 0, 0);
        }
      }
    }
  };
  // the stream's BF16 rounding, position-major: 4 consecutive channels per write
  auto publish = [&] {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        bf16x4 v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = to_bf16(h[i][j][q]);
        *reinterpret_cast<bf16x4*>(&Hs[16 * j + lr][net_col((wv * RT + i) * 16 + 4 * g)]) = v;
      }
  };

  // embedding: its output, or formed here
  int row[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) row[j] = 16 * j + lr;
  if constexpr (!kEmbed) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float* src = a.h0 + ((wv * RT + i) * 16 + 4 * g + q) * N + p0;
#pragma unroll
        for (int j = 0; j < NT; ++j) h[i][j][q] = p0 + row[j] < N ? src[row[j]] : 0.f;
      }
  } else {
    // column blocks of C of the reduction, of whole (sine, cosine) pairs: one
    // block, or 2 P divides C
    const int Kr = 2 * a.ny * a.P, se = net_steps(Kr);
    clear();
    for (int kb = 0; kb < Kr; kb += C) {
      const int cols = min(C, 32 * (se - kb / 32)), per = min(C, Kr - kb) / 2;
      const int s0 = kb / (2 * a.P), ns = per / a.P;   // first sensor of the block, sensors in it
      if (kb > 0) __syncthreads();
      // columns past the reduction of the last step
      for (int e = t; e < kNetP * 32; e += 256) {
        const int c = cols - 32 + (e & 31);
        if (kb + c >= Kr) Hs[e >> 5][net_col(c)] = 0;
      }
      for (int e = t; e < kNetP * per; e += 256) {
        const int p = e / per, q = e - p * per, s = q % ns, k = q / ns;
        const int c0 = 2 * s * a.P + k, c1 = c0 + a.P;   // sine, cosine columns
        float sf = 0.f, cf = 0.f;
        if (p0 + p < N) {
          const int64_t w = a.w0 + (p0 + p) / a.Lpos;
          const int tr = a.tab.track[w];
          const int64_t m0 = a.tab.meas_off[tr], T = a.tab.meas_off[tr + 1] - m0;
          const int64_t st = min(int64_t(a.tab.start[w]) + ((p0 + p) % a.Lpos) * a.P + k, T);
          double sv, cv;
          sincos(a.y[(m0 + st - 1) * a.ny + s0 + s], &sv, &cv);
          sf = float(sv);
          cf = float(cv);
        }
        Hs[p][net_col(c0)] = to_bf16(sf);
        Hs[p][net_col(c1)] = to_bf16(cf);
      }
      __syncthreads();
      product(a.we, se, kb / 32, cols / 32, row);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float b = a.be[(wv * RT + i) * 16 + 4 * g + q];
#pragma unroll
        for (int j = 0; j < NT; ++j) h[i][j][q] = fmaxf(acc[i][j][q] + b, 0.f);
      }
  }
  __syncthreads();
  publish();
  __syncthreads();

  // residual layers: h += relu(b + sum over taps)
  constexpr int SC = C / 32;
  for (int l = 0; l < a.hidden; ++l) {
    const short* w = a.wr + int64_t(l) * net_words(C, 3 * C);
    const int dil = 1 << l;
    clear();
    for (int k = 0; k < 3; ++k) {
      const int off = (k - 1) * dil;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int pl = 16 * j + lr, q = pl % a.Lpos + off;
        row[j] = q >= 0 && q < a.Lpos ? pl + off : kNetP;
      }
      product(w, 3 * SC, k * SC, SC, row);
    }
    const float* bias = a.br + l * a.br_stride;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float b = bias[(wv * RT + i) * 16 + 4 * g + q];
#pragma unroll
        for (int j = 0; j < NT; ++j) h[i][j][q] += fmaxf(acc[i][j][q] + b, 0.f);
      }
    __syncthreads();
    publish();
    __syncthreads();
  }

  if constexpr (!kHead) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float* dst = a.h1 + ((wv * RT + i) * 16 + 4 * g + q) * N + p0;
#pragma unroll
        for (int j = 0; j < NT; ++j)
          if (p0 + 16 * j + lr < N) dst[16 * j + lr] = h[i][j][q];
      }
    return;
  }

  // head: each wave takes 32 positions and every output row; step k of a track
  // comes from window min((k - 1) / W, n_w - 1) of it, slot 0 from step 1
  const int M = a.P * a.nx;
  for (int mt = 0; mt * 16 < M; ++mt) {
    f32x4 o[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int s = 0; s < SC; ++s) {
      const bf16x8 af = *reinterpret_cast<const bf16x8*>(a.wh + (int64_t(mt) * SC + s) * 512 + ln * 8);
      const bf16x4 a0 = __builtin_shufflevector(af, af, 0, 1, 2, 3), a1 = __builtin_shufflevector(af, af, 4, 5, 6, 7);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(&Hs[32 * wv + 16 * j + lr][32 * s + 8 * g]);
        const bf16x4 b0 = __builtin_shufflevector(b, b, 0, 1, 2, 3), b1 = __builtin_shufflevector(b, b, 4, 5, 6, 7);
        o[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, b0, o[j], 0, 0, 0);
        o[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, b1, o[j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t p = p0 + 32 * wv + 16 * j + lr;
      if (p >= N) continue;
      const int64_t w = a.w0 + p / a.Lpos;
      const int tr = a.tab.track[w];
      const int64_t m0 = a.tab.meas_off[tr], T = a.tab.meas_off[tr + 1] - m0;
      const int64_t k0 = int64_t(a.tab.start[w]) + (p % a.Lpos) * a.P;
      const int first = a.tab.first[tr], nw = a.tab.first[tr + 1] - first;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = mt * 16 + 4 * g + q;
        if (m >= M) continue;
        const int u = m / a.nx, i = m - u * a.nx;
        const int64_t k = k0 + u;
        if (k > T || first + min((k - 1) / a.W, int64_t(nw - 1)) != w) continue;
        const float out = o[j][q] + a.bh[m];
        const double v = double(a.mu[i] + a.sigma[i] * out);
        double* x = a.mean + (m0 + tr + k) * a.nx + i;
        *x = v;
        if (k == 1) x[-a.nx] = v;
      }
    }
  }
}

}  // namespace wsn
