// Device side of the stress surrogate (gfx950): one LDS-staged BF16 matrix-core GEMM with fused
// epilogues, and the small kernels around it (normalisation, loss, bias gradients, Adam,
// ensemble statistics).  All padded dimensions are multiples of 64; padded rows and columns
// carry zeros (inputs, weights, output gradients), so they never contribute.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rsur {

typedef __bf16 bf16;
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

enum Epi : int { EPI_FWD_HIDDEN = 0, EPI_FWD_OUT = 1, EPI_BWD_DA = 2, EPI_BWD_DW = 3 };

struct GemmArgs {
  const bf16* A; long long lda, sA;        // operand A, row stride, member stride
  const bf16* B; long long ldb, sB;
  int M, N, K;                             // C is M x N, reduction over K (multiples of 64, K / ksplit too)
  const float* bias; long long sBias;
  float* Z; long long ldz, sZ;             // FP32 result (pre-activation, output or gradient)
  bf16* O; long long ldo, sO;              // BF16 result (activation or backpropagated gradient)
  const float* Zp; long long ldzp, sZp;    // pre-activation whose SiLU derivative scales the result
  int nmem, ksplit;                        // members; reduction ranges (weight gradient only, else 1)
  long long sRange;                        // ksplit > 1: distance of the ranges' partial results in Z and colsum
  float* colsum; long long sCol;           // weight gradient: column sums of B (the bias gradient) go here too
};

constexpr int COL_G = 16;          // partial sums per column of the bias gradient (four waves of four)
constexpr int TM = 64, TN = 64, TK = 64, LDK = 72;   // tile sizes; LDS row stride padded to 72

// An operand tile on its way to LDS: 64 rows of the output dimension by TK of the reduction, two 16-byte
// pieces per thread of 256.  Direct: rows of consecutive k.  Transposed: consecutive k-rows in pairs, so that
// two k of a column leave as one 4-byte store, 32 of them side by side in a wave (single elements, eight
// lanes to a bank, before).
template <bool DIRECT>
struct TileLoad {
  v8bf v[2];
  __device__ void request(const bf16* p, long long ld, int o0, int k0, int t) {
    if constexpr (DIRECT) {
      const int r = t >> 2, c = (t & 3) * 16;
      const bf16* q = p + (long long)(o0 + r) * ld + k0 + c;
      v[0] = *(const v8bf*)q; v[1] = *(const v8bf*)(q + 8);
    } else {
      const int r = 2 * (t & 31), c = (t >> 5) * 8;
      const bf16* q = p + (long long)(k0 + r) * ld + o0 + c;
      v[0] = *(const v8bf*)q; v[1] = *(const v8bf*)(q + ld);
    }
  }
  __device__ void store(bf16* s, int t) const {
    if constexpr (DIRECT) {
      const int r = t >> 2, c = (t & 3) * 16;
      *(v8bf*)&s[r * LDK + c] = v[0]; *(v8bf*)&s[r * LDK + c + 8] = v[1];
    } else {
      const int r = 2 * (t & 31), c = (t >> 5) * 8;
#pragma unroll
      for (int q = 0; q < 8; ++q) *(v2bf*)&s[(c + q) * LDK + r] = (v2bf){v[0][q], v[1][q]};
    }
  }
};

__device__ __forceinline__ float silu(float z) { return z / (1.0f + __expf(-z)); }
__device__ __forceinline__ float silu_grad(float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return s * (1.0f + z * (1.0f - s));
}

// C(m, n) = sum_k A(m, k) B(k, n) for member blockIdx.z, with A(m, k) = A[m lda + k] (or
// A[k lda + m] when AT) and B(k, n) = B[k ldb + n] (or B[n ldb + k] when BT).  A 256-thread block
// computes a 64 x 64 tile: four waves of 32 x 32, each accumulating v_mfma_f32_32x32x16_bf16
// products over K in steps of TK staged through LDS as [m][k] and [n][k] rows, the next step's pieces
// requested before this step's products.  The products are small (256 wide): bound by the traffic of
// the activations and FP32 pre-activations, ~8 us per layer of 4096 rows and 5 members at 5 TB/s.
// Measured at that size, TK = 32 and no request ahead / now: forward 19.4 / 15.9 us, output gradient
// 12.3 / 11.4, weight gradient 24.8 (its transposed tiles stored to LDS element by element) / 13.4
// including the column sums, which took 9.7 in a kernel of their own.
struct GemmLds { __attribute__((aligned(16))) bf16 a[TM * LDK], b[TN * LDK]; };
template <bool AT, bool BT, int EPI>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, int m0, int n0, int z, GemmLds& sh) {
  bf16 *sa = sh.a, *sb = sh.b;
  // z = member + nmem * range: the weight gradient's reduction over the batch is split
  // into ksplit consecutive ranges of K / ksplit (a multiple of TK), each block taking one
  const int mem = z % g.nmem, ks = z / g.nmem;
  const int kc = g.K / g.ksplit;
  const bf16* A = g.A + mem * g.sA;
  const bf16* B = g.B + mem * g.sB;
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  v16f acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  // the first row of blocks of the weight gradient adds up the columns of B as they pass by: wave w takes
  // the rows k with k % COL_G in [4 w, 4 w + 4), a sum each, lane l column n0 + l
  const bool cols = EPI == EPI_BWD_DW && m0 == 0;
  float col_acc[4] = {0, 0, 0, 0};
  TileLoad<!AT> la;
  TileLoad<BT> lb;
  la.request(A, g.lda, m0, ks * kc, t);
  lb.request(B, g.ldb, n0, ks * kc, t);
  for (int k0 = ks * kc; k0 < (ks + 1) * kc; k0 += TK) {
    la.store(sa, t);
    lb.store(sb, t);
    __syncthreads();
    if (k0 + TK < (ks + 1) * kc) {
      la.request(A, g.lda, m0, k0 + TK, t);
      lb.request(B, g.ldb, n0, k0 + TK, t);
    }
#pragma unroll
    for (int s = 0; s < TK; s += 16) {
      const v8bf a = *(const v8bf*)&sa[(wm + (l & 31)) * LDK + s + 8 * (l >> 5)];
      const v8bf b = *(const v8bf*)&sb[(wn + (l & 31)) * LDK + s + 8 * (l >> 5)];
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
    if constexpr (EPI == EPI_BWD_DW) {
      if (cols)
#pragma unroll
        for (int k = 0; k < TK; k += COL_G) {
          const v4bf v = *(const v4bf*)&sb[l * LDK + k + 4 * w];
#pragma unroll
          for (int q = 0; q < 4; ++q) col_acc[q] += (float)v[q];
        }
    }
    __syncthreads();
  }
  if constexpr (EPI == EPI_BWD_DW) {
    if (cols) {
      float* red = (float*)sa;                   // [COL_G][TN]; the products have been read
#pragma unroll
      for (int q = 0; q < 4; ++q) red[(4 * w + q) * TN + l] = col_acc[q];
      __syncthreads();
      if (t < TN) {
        float v = 0.0f;
        for (int r = 0; r < COL_G; ++r) v += red[r * TN + t];
        g.colsum[ks * g.sRange + mem * g.sCol + n0 + t] = v;
      }
    }
  }
  // accumulator element r of lane l holds C(row, col) with the row below
  const int col = n0 + wn + (l & 31);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const long long row = m0 + wm + (r >> 2) * 8 + (l >> 5) * 4 + (r & 3);
    const float v = acc[r];
    if (EPI == EPI_FWD_HIDDEN) {
      const float z = v + g.bias[mem * g.sBias + col];
      g.Z[mem * g.sZ + row * g.ldz + col] = z;
      g.O[mem * g.sO + row * g.ldo + col] = (bf16)silu(z);
    } else if (EPI == EPI_FWD_OUT) {
      g.Z[mem * g.sZ + row * g.ldz + col] = v + g.bias[mem * g.sBias + col];
    } else if (EPI == EPI_BWD_DA) {
      g.O[mem * g.sO + row * g.ldo + col] = (bf16)(v * silu_grad(g.Zp[mem * g.sZp + row * g.ldzp + col]));
    } else {
      g.Z[ks * g.sRange + mem * g.sZ + row * g.ldz + col] = v;
    }
  }
}

template <bool AT, bool BT, int EPI>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs g) {
  __shared__ GemmLds sh;
  gemm_tile<AT, BT, EPI>(g, blockIdx.y * TM, blockIdx.x * TN, blockIdx.z, sh);
}

constexpr int MAXL = 8;            // most layers of the fused kernels
// The weight gradients of all layers in one launch: 64 tiles of five members in 8 ranges are 2560 blocks, one
// launch of them without the gaps and half-empty ends of five: 51 us for 4096 rows, 67 in five launches.
// Latency and the L2 bound it: parts of 32 x 64 per wave, with a quarter fewer LDS reads, took the same 51 us, and
// the tiles of one member and range placed on one XCD 48.
struct DwArgs { GemmArgs g[MAXL]; int first[MAXL + 1]; };   // layer l: tiles first[l] ... first[l + 1]
__global__ __launch_bounds__(256) void k_dw(DwArgs d) {
  __shared__ GemmLds sh;
  int l = 0;
  while ((int)blockIdx.x >= d.first[l + 1]) ++l;
  const int e = blockIdx.x - d.first[l], nx = d.g[l].N / TN;
  gemm_tile<true, false, EPI_BWD_DW>(d.g[l], e / nx * TM, e % nx * TN, blockIdx.y, sh);
}

// ------------------------------------------------------------------ fused inference and training pass
// Every layer of one member for 32 RT rows in one block of NW waves: the activations stay in LDS (one
// buffer, overwritten in place between two barriers per layer) and the first layer normalises the raw
// inputs itself.  A wave computes the transposed product: 32 output features of the weights (operand A)
// by 32 rows of activations (operand B) per v_mfma_f32_32x32x16_bf16, so an accumulator's four
// consecutive registers are four consecutive features of one row - one 8-byte LDS store after the
// activation, where the row-major product took four 2-byte ones.  Over k in steps of 16 from zero, the
// order of k_gemm, so the outputs equal the layer-wise forward bit for bit.
//
// The weights come from a copy laid out by fragments (frag_index): the 64 lanes of a wave read one
// operand as 1 KB of consecutive memory (a transposed copy gave 32 pieces of 32 bytes).  They are read
// once per block, so the large variant takes 128 rows per block (64 before); the small one spreads 32
// rows over 8 waves and requests a layer's whole operand at once, since a small batch waits for latency.
//
// Bound: per block of 128 rows the matrix products take ~16 000 cycles of every SIMD (32 each) and SiLU
// ~25 000 (12 instructions, two of them transcendental, per 64 elements); two blocks per CU run them side by
// side.  Measured (one MI355X, 153 -> 4 x 256 -> 6, 5 members), this kernel alone, traced, which slows it: 60 001 rows
// 266 us, 683 with 64 rows per block, a transposed weight copy, a full division and inputs normalised one load at a
// time (four waves of two tiles instead of eight of one 13 % more); 256 rows 15.8 us, ~44 layer by layer in six
// launches.  Untraced, with the ensemble mean behind it, a call among others takes 214-224 and 8.6 us.
constexpr int FW = 256, FLD = FW + 8;

struct MlpArgs {
  const float* X; int B, din;
  const float *xmu, *xsd;
  const bf16* wf; long long sW;              // BF16 weights by fragments, member stride
  const float* p; long long sP;              // FP32 parameters (biases), member stride
  int L, dout;
  int dp[MAXL + 1];
  long long woff[MAXL], boff[MAXL];
  float* out; long long sOut; int ldo;       // K x Mp x dp[L]
};

// Element offset of weight (k, n) in a layer's fragment copy: features in tiles of 32, k in steps of 16;
// lane l of a fragment holds feature l % 32 and the 8 consecutive k from 8 (l / 32).
__host__ __device__ inline long long frag_index(int k, int n, int Kd) {
  const int lane = (n & 31) + 32 * ((k >> 3) & 1);
  return (((long long)(n >> 5) * (Kd >> 4) + (k >> 4)) * 64 + lane) * 8 + (k & 7);
}

// z / (1 + e^-z), the quotient rounded as by a division: the residual of a first quotient, exact by a
// fused multiply-add, corrects it.  A non-finite z, or one so negative that e^-z overflows, gives NaN
// here: the caller redoes those by silu().
__device__ __forceinline__ float silu_fast(float z) {
  const float d = 1.0f + __builtin_amdgcn_exp2f(z * -1.442695041f);
  const float r = __builtin_amdgcn_rcpf(d), q = z * r;
  return fmaf(fmaf(-d, q, z), r, q);
}

// The training pass keeps going where inference ends: the block turns its outputs into their gradient and
// walks the layers back with the transposed weights (their own copy by fragments).  Activations and output
// gradients are written row by row for the weight gradients; a pre-activation is read again by the lane
// that wrote it, so these go out and come in as whole accumulators, 1 KB per wave and access.  Layer by layer
// every product read its input and the pre-activations in rows and wrote them again.  Bound by memory: 4096
// rows of 5 members move 260 MB, 50 us at 5.2 TB/s; 76 us (64 rows per block), 131 and the gaps between 11
// launches before.
struct TrainArgs {
  const float *Y, *ymu, *ysd;
  const bf16* wt;                            // BF16 transposed weights by fragments, member stride sW
  bf16* act[MAXL];                           // normalised input and activations
  // Pre-activations in accumulator order, then (and for the output layer from the first) the layer's output
  // gradient: 32 rows of either lie in the same bytes, a row of the gradient in the first half of its share, and
  // a block has read its pre-activations before it writes there.
  float* Z[MAXL];
  float* lpart;                              // [member][block] squared-error sums
  int Mp, rows;                              // padded rows of this batch; rows of a member in the buffers
  float inv;
};

// rows of a block's LDS buffer to / from memory, dp <= FW columns, rows of ld in memory, two rows per wave at a time
template <int ROWS, int NW, bool OUT>
__device__ __forceinline__ void mlp_rows(bf16* lds, bf16* mem, int dp, int ld, int nrows) {
  const int l = threadIdx.x & 63, k = 8 * (l & 31);
  for (int r = 2 * (threadIdx.x >> 6) + (l >> 5); r < ROWS; r += 2 * NW) {
    if (k >= dp) continue;
    if constexpr (OUT) {
      if (r < nrows) *(v8bf*)(mem + (long long)r * ld + k) = *(const v8bf*)(lds + r * FLD + k);
    } else {
      v8bf v = {};
      if (r < nrows) v = *(const v8bf*)(mem + (long long)r * ld + k);
      *(v8bf*)(lds + r * FLD + k) = v;
    }
  }
}

// SiLU'(z) with the logistic function as silu_fast's quotient; NaN where that is
__device__ __forceinline__ float silu_grad_fast(float z) {
  const float d = 1.0f + __builtin_amdgcn_exp2f(z * -1.442695041f);
  const float r = __builtin_amdgcn_rcpf(d), s = fmaf(fmaf(-d, r, 1.0f), r, r);
  return s * (1.0f + z * (1.0f - s));
}

template <int RT, int NW, bool TRAIN>
__device__ __forceinline__ void mlp_block(const MlpArgs& g, const TrainArgs& h, bf16* act) {
  // FT feature tiles per wave at most: one with the eight waves of every instance.  (Without the loops over f
  // k_mlp_train<1, 8> takes 134 registers instead of 118, and a CU holds one block of it instead of two.)
  constexpr int ROWS = 32 * RT, FT = (FW / 32) / NW;
  const int mem = blockIdx.y, m0 = blockIdx.x * ROWS;
  const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63;
  const int lr = l & 31, lk = 8 * (l >> 5), lf = 4 * (l >> 5);
  const bf16* Wm = g.wf + mem * g.sW;
  const float* Pm = g.p + mem * g.sP;
  // RT = 1: a layer's whole operand of this wave, requested while the layer before is being activated
  constexpr int KM = RT == 1 ? FW / 16 : 1;
  v8bf pre[FT][KM];
  auto request_operand = [&](const bf16* W, int KS, int NF) {
    const bf16* W0 = W + ((long long)w * KS * 64 + l) * 8;
#pragma unroll
    for (int k = 0; k < KM; ++k)
#pragma unroll
      for (int f = 0; f < FT; ++f)
        if (k < KS && w + NW * f < NF) pre[f][k] = *(const v8bf*)(W0 + ((long long)NW * f * KS + k) * 512);
  };
  auto request_layer = [&](int L) {
    request_operand(Wm + g.woff[L], g.dp[L] >> 4, L + 1 < g.L ? g.dp[L + 1] >> 5 : (g.dout + 31) >> 5);
  };
  if constexpr (RT == 1) request_layer(0);
  // normalised inputs: a lane keeps its column's statistics and has RB rows' loads on the way at once (row
  // by row, this took 77 000 of a block's 200 000 cycles)
  constexpr int WROWS = ROWS / NW, RB = WROWS < 16 ? WROWS : 16;
  for (int k = l; k < g.dp[0]; k += 64) {
    const int kc = min(k, g.din - 1);
    const float mu = g.xmu[kc], sd = g.xsd[kc];
#pragma unroll
    for (int r0 = 0; r0 < WROWS; r0 += RB) {
      float x[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) x[r] = g.X[(long long)min(m0 + w * WROWS + r0 + r, g.B - 1) * g.din + kc];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const int row = w * WROWS + r0 + r;
        act[row * FLD + k] = (m0 + row < g.B && k < g.din) ? (bf16)((x[r] - mu) / sd) : (bf16)0.0f;
      }
    }
  }
  __syncthreads();
  const bf16* arow = act + lr * FLD + lk;
  // acc = the product of one layer: KS steps of 16 over the rows in LDS, NF feature tiles
  auto product = [&](v16f (&acc)[FT][RT], const bf16* W, int KS, int NF) {
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
      for (int c = 0; c < RT; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[f][c][r] = 0.0f;
    // feature tiles w, w + NW, ...; a layer narrower than the block leaves its last waves idle
    const bf16* W0 = W + ((long long)w * KS * 64 + l) * 8;
    const long long wstep = (long long)NW * KS * 512;
    if (w < NF) {
      if constexpr (RT == 1) {
#pragma unroll
        for (int k = 0; k < KM; ++k)
          if (k < KS) {
            const v8bf b = *(const v8bf*)(arow + 16 * k);
#pragma unroll
            for (int f = 0; f < FT; ++f)
              if (w + NW * f < NF) acc[f][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pre[f][k], b, acc[f][0], 0, 0, 0);
          }
      } else {
        // the operands of four steps ahead: 32 products (1024 cycles) cover their way from the L2
        const bool two = FT > 1 && w + NW < NF;     // uniform: the wave has all its tiles, or the first alone
        v8bf a[2][4][FT];
        auto request = [&](v8bf (&to)[4][FT], int k) {
#pragma unroll
          for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int f = 0; f < FT; ++f)
              if (f == 0 || two) to[h][f] = *(const v8bf*)(W0 + f * wstep + (k + h) * 512);
        };
        auto steps = [&](const v8bf (&from)[4][FT], int k) {
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            v8bf b[RT];
#pragma unroll
            for (int c = 0; c < RT; ++c) b[c] = *(const v8bf*)(arow + c * 32 * FLD + 16 * (k + h));
#pragma unroll
            for (int f = 0; f < FT; ++f)
              if (f == 0 || two)
#pragma unroll
                for (int c = 0; c < RT; ++c)
                  acc[f][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(from[h][f], b[c], acc[f][c], 0, 0, 0);
          }
        };
        request(a[0], 0);                           // KS is a multiple of 4 (padded widths are of 64)
        for (int k = 0; k < KS; k += 8) {
          if (k + 4 < KS) request(a[1], k + 4);
          steps(a[0], k);
          if (k + 4 < KS) {
            if (k + 8 < KS) request(a[0], k + 8);
            steps(a[1], k + 4);
          }
        }
      }
    }
  };
  const int nrows = min(ROWS, h.Mp - m0);        // training: rows of this block that the buffers hold
#pragma unroll 1                                 // peeled, the kernel misses the instruction cache: 8.6 / 10.8 us for 256 rows
  for (int L = 0; L < g.L - 1; ++L) {
    const int NF = g.dp[L + 1] >> 5;
    if constexpr (TRAIN)                         // this layer's input, the network's (alike for all members) once
      if (L > 0 || mem == 0)
        mlp_rows<ROWS, NW, true>(act, h.act[L] + (L > 0 ? mem * (long long)h.rows * g.dp[L] : 0) + (long long)m0 * g.dp[L],
                                 g.dp[L], g.dp[L], nrows);
    v16f acc[FT][RT];
    product(acc, Wm + g.woff[L], g.dp[L] >> 4, NF);
    if constexpr (TRAIN) {
      float* Z = h.Z[L] + mem * (long long)h.rows * g.dp[L + 1] + 4 * l;
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        const int ft = w + NW * f;
        if (ft >= NF) break;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 bias = *(const float4*)(Pm + g.boff[L] + 32 * ft + 8 * q + lf);
#pragma unroll
          for (int c = 0; c < RT; ++c) {
            acc[f][c][4 * q] += bias.x; acc[f][c][4 * q + 1] += bias.y;
            acc[f][c][4 * q + 2] += bias.z; acc[f][c][4 * q + 3] += bias.w;
            if (32 * c < nrows)
              *(float4*)(Z + (((long long)(m0 >> 5) + c) * NF + ft) * 1024 + q * 256) =
                  make_float4(acc[f][c][4 * q], acc[f][c][4 * q + 1], acc[f][c][4 * q + 2], acc[f][c][4 * q + 3]);
          }
        }
      }
    }
    if constexpr (RT == 1) request_layer(L + 1);
    __syncthreads();                             // every wave has read this layer's input
    auto activate = [&](auto&& fn) {             // features 32 ft + 8 q + lf + 0..3 of row 32 c + lr
#pragma unroll
      for (int f = 0; f < FT; ++f) {
        const int ft = w + NW * f;
        if (ft >= NF) break;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int n = 32 * ft + 8 * q + lf;
          const float4 bias = TRAIN ? make_float4(0, 0, 0, 0) : *(const float4*)(Pm + g.boff[L] + n);
#pragma unroll
          for (int c = 0; c < RT; ++c) {
            const v4bf o = {(bf16)fn(acc[f][c][4 * q] + bias.x), (bf16)fn(acc[f][c][4 * q + 1] + bias.y),
                            (bf16)fn(acc[f][c][4 * q + 2] + bias.z), (bf16)fn(acc[f][c][4 * q + 3] + bias.w)};
            *(v4bf*)(act + (32 * c + lr) * FLD + n) = o;
          }
        }
      }
    };
    float bad = 0.0f;                            // NaN once any result is
    activate([&](float z) { const float y = silu_fast(z); bad = fmaf(y, 0.0f, bad); return y; });
    if (__any(!(bad == 0.0f))) activate([](float z) { return silu(z); });
    __syncthreads();
  }
  // the linear output: only the tiles that hold real outputs, shared out by row tiles
  const int KS = g.dp[g.L - 1] >> 4, NF = (g.dout + 31) >> 5, dpo = g.dp[g.L];
  if constexpr (TRAIN)
    if (g.L > 1 || mem == 0)
      mlp_rows<ROWS, NW, true>(act, h.act[g.L - 1] + (g.L > 1 ? mem * (long long)h.rows * g.dp[g.L - 1] : 0) +
                               (long long)m0 * g.dp[g.L - 1], g.dp[g.L - 1], g.dp[g.L - 1], nrows);
  const int ldo = 2 * dpo;                       // rows of the output gradient
  bf16* dzo = TRAIN ? (bf16*)h.Z[g.L - 1] + (mem * (long long)h.rows + m0) * ldo : nullptr;
  float sq = 0.0f;                               // training: squared errors of this lane
  for (int it = w; it < (TRAIN ? dpo >> 5 : NF) * RT; it += NW) {
    const int ft = it / RT, c = it % RT;
    if (TRAIN && ft >= NF) {                     // padding columns
      if (32 * c < nrows)
#pragma unroll
        for (int q = 0; q < 4; ++q) *(v4bf*)(dzo + (32 * c + lr) * ldo + 32 * ft + 8 * q + lf) = (v4bf){};
      continue;
    }
    const bf16* W0 = Wm + g.woff[g.L - 1] + ((long long)ft * KS * 64 + l) * 8;
    v16f acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    if constexpr (RT == 1) {                     // tile `it` is this wave's: NF <= NW
#pragma unroll
      for (int k = 0; k < KM; ++k)
        if (k < KS) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pre[0][k], *(const v8bf*)(arow + 16 * k), acc, 0, 0, 0);
    } else {
#pragma unroll 4
      for (int k = 0; k < KS; ++k)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const v8bf*)(W0 + k * 512), *(const v8bf*)(arow + c * 32 * FLD + 16 * k), acc, 0, 0, 0);
    }
    const int m = m0 + 32 * c + lr;
    if constexpr (TRAIN) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        v4bf d = {};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = 32 * ft + 8 * q + lf + e;
          if (m >= g.B || n >= g.dout) continue;
          const float yn = (h.Y[(long long)m * g.dout + n] - h.ymu[n]) / h.ysd[n];
          const float r = acc[4 * q + e] + Pm[g.boff[g.L - 1] + n] - yn;
          sq += r * r;
          d[e] = (bf16)(2.0f * r * h.inv);
        }
        if (32 * c < nrows) *(v4bf*)(dzo + (32 * c + lr) * ldo + 32 * ft + 8 * q + lf) = d;
      }
    } else if (m < g.B) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = 32 * ft + 8 * q + lf;
        if (n < g.dout) {
          const float4 bias = *(const float4*)(Pm + g.boff[g.L - 1] + n);
          *(float4*)(g.out + mem * g.sOut + (long long)m * g.ldo + n) =
              make_float4(acc[4 * q] + bias.x, acc[4 * q + 1] + bias.y, acc[4 * q + 2] + bias.z, acc[4 * q + 3] + bias.w);
        }
      }
    }
  }
  if constexpr (TRAIN) {
    if constexpr (RT == 1)
      if (g.L > 1) request_operand(h.wt + mem * g.sW + g.woff[g.L - 1], dpo >> 4, g.dp[g.L - 1] >> 5);
    __shared__ float sums[NW];
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
    if (l == 0) sums[w] = sq;
    __syncthreads();                             // the output gradient is written, the last input read
    if (t == 0) {
      float v = 0.0f;
      for (int q = 0; q < NW; ++q) v += sums[q];
      h.lpart[(long long)mem * gridDim.x + blockIdx.x] = v;
    }
    if (g.L > 1) mlp_rows<ROWS, NW, false>(act, dzo, dpo, ldo, nrows);
    __syncthreads();
#pragma unroll 1
    for (int L = g.L - 1; L >= 1; --L) {         // dZ_{L-1} = (dZ_L W_L^T) * SiLU'(Z_{L-1})
      const int NF = g.dp[L] >> 5;
      const float* Z = h.Z[L - 1] + mem * (long long)h.rows * g.dp[L] + 4 * l;
      float4 z[FT][RT][4];                       // on their way while the product is computed
#pragma unroll
      for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int c = 0; c < RT; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (w + NW * f < NF && 32 * c < nrows)
              z[f][c][q] = *(const float4*)(Z + (((long long)(m0 >> 5) + c) * NF + w + NW * f) * 1024 + q * 256);
      v16f acc[FT][RT];
      product(acc, h.wt + mem * g.sW + g.woff[L], g.dp[L + 1] >> 4, NF);
      if constexpr (RT == 1)
        if (L > 1) request_operand(h.wt + mem * g.sW + g.woff[L - 1], g.dp[L] >> 4, g.dp[L - 1] >> 5);
      __syncthreads();                           // every wave has read dZ_L
      auto back = [&](auto&& fn) {
#pragma unroll
        for (int f = 0; f < FT; ++f) {
          const int ft = w + NW * f;
          if (ft >= NF) break;
#pragma unroll
          for (int c = 0; c < RT; ++c) {
            if (32 * c >= nrows) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const float4 y = z[f][c][q];
              const v4bf o = {(bf16)(acc[f][c][4 * q] * fn(y.x)), (bf16)(acc[f][c][4 * q + 1] * fn(y.y)),
                              (bf16)(acc[f][c][4 * q + 2] * fn(y.z)), (bf16)(acc[f][c][4 * q + 3] * fn(y.w))};
              *(v4bf*)(act + (32 * c + lr) * FLD + 32 * ft + 8 * q + lf) = o;
            }
          }
        }
      };
      float bad = 0.0f;
      back([&](float y) { const float d = silu_grad_fast(y); bad = fmaf(d, 0.0f, bad); return d; });
      if (__any(!(bad == 0.0f))) back([](float y) { return silu_grad(y); });
      __syncthreads();
      mlp_rows<ROWS, NW, true>(act, (bf16*)h.Z[L - 1] + (mem * (long long)h.rows + m0) * 2 * g.dp[L], g.dp[L], 2 * g.dp[L], nrows);
    }
  }
}

template <int RT, int NW>
__global__ __launch_bounds__(64 * NW, RT == 1 ? 2 : 4) void k_mlp_forward(MlpArgs g) {
  __shared__ __attribute__((aligned(16))) bf16 act[32 * RT * FLD];
  mlp_block<RT, NW, false>(g, TrainArgs{}, act);
}
template <int RT, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_mlp_train(MlpArgs g, TrainArgs h) {
  __shared__ __attribute__((aligned(16))) bf16 act[32 * RT * FLD];
  mlp_block<RT, NW, true>(g, h, act);
}

struct FragMap { int L; int dp[MAXL + 1]; long long woff[MAXL]; };   // L = 0: no fragment copy
// parameter o of the member at `base` in BF16, and a weight into its copies by fragments
__device__ __forceinline__ void store_bf16(bf16* pb, bf16* pbf, bf16* pbt, const FragMap& map, long long base, long long o, float w) {
  pb[base + o] = (bf16)w;
  for (int l = 0; l < map.L; ++l) {
    const long long r = o - map.woff[l];
    if (r < 0 || r >= (long long)map.dp[l] * map.dp[l + 1]) continue;
    const int k = (int)r / map.dp[l + 1], n = (int)r - k * map.dp[l + 1];
    pbf[base + map.woff[l] + frag_index(k, n, map.dp[l])] = (bf16)w;
    pbt[base + map.woff[l] + frag_index(n, k, map.dp[l + 1])] = (bf16)w;
  }
}
// every parameter of the member at `base`, in one launch: rsur_set_params of 153 -> 4 x 256 -> 6 takes 176 us, 199 with a
// launch more per layer for the copies
__global__ void k_to_bf16(const float* p, bf16* pb, bf16* pbf, bf16* pbt, FragMap map, long long P, long long base) {
  const long long o = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (o < P) store_bf16(pb, pbf, pbt, map, base, o, p[base + o]);
}

// raw inputs (B x din, FP32) -> normalised BF16 rows of width dp0, zero padding
__global__ void k_norm_in(const float* X, int B, int din, int Mp, int dp0, const float* mu, const float* sd, bf16* out) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)Mp * dp0) return;
  const int m = (int)(e / dp0), k = (int)(e % dp0);
  out[e] = (m < B && k < din) ? (bf16)((X[(long long)m * din + k] - mu[k]) / sd[k]) : (bf16)0.0f;
}

// MSE on normalised outputs and its output gradient: block (chunk, member) takes LOSS_ROWS rows of one
// member and writes its squared-error sum to part[member][chunk] (a fixed tree over the block);
// k_loss_total adds the chunks in order.  (16 chunks per member left most of the GPU idle: 31 us at 4096
// rows, 9.8 now.)  Element indices are 64-bit (Mp * ldo may exceed 2^31).
constexpr int LOSS_NT = 256, LOSS_ROWS = 64;
__global__ __launch_bounds__(LOSS_NT) void k_loss(const float* out, long long sOut, int ldo, const float* Y, int B,
                                                  int dout, const float* ymu, const float* ysd, bf16* dY,
                                                  long long sdY, float* part) {
  __shared__ float sh[LOSS_NT];
  const int chunk = blockIdx.x, mem = blockIdx.y;
  const float inv = 1.0f / ((float)B * (float)dout);
  float acc = 0.0f;
  // a row's columns 64 at a time, so that a wave stays in one row
  for (int r = threadIdx.x >> 6; r < LOSS_ROWS; r += LOSS_NT / 64) {
    const long long m = (long long)chunk * LOSS_ROWS + r;
    for (int n = threadIdx.x & 63; n < ldo; n += 64) {
      float gr = 0.0f;
      if (m < B && n < dout) {
        const float yn = (Y[m * dout + n] - ymu[n]) / ysd[n];
        const float d = out[mem * sOut + m * ldo + n] - yn;
        acc += d * d;
        gr = 2.0f * d * inv;
      }
      dY[mem * sdY + m * ldo + n] = (bf16)gr;
    }
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int s = LOSS_NT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[(long long)mem * gridDim.x + chunk] = sh[0];
}

// one wave per member: lane q adds the chunks q, q + 64, ... in order, then the lanes in order
__global__ __launch_bounds__(64) void k_loss_total(const float* part, int chunks, float inv, float* loss) {
  __shared__ float sh[64];
  const int mem = blockIdx.x;
  float t = 0.0f;
  for (int c = threadIdx.x; c < chunks; c += 64) t += part[(long long)mem * chunks + c];
  sh[threadIdx.x] = t;
  __syncthreads();
  if (threadIdx.x != 0) return;
  t = 0.0f;
  for (int q = 0; q < 64; ++q) t += sh[q];
  loss[mem] = t * inv;
}

// Adam on every padded parameter of every member: the gradient is the sum, in order, of the S ranges'
// partial sums (S = 1: gr itself); refreshes the BF16 weights and their copies by fragments.  Padding
// stays zero: its gradient is zero.  Bound by memory: 8 ranges of 5 x 263 000 parameters are 85 MB in and
// out, 19.7 us (9 us before, and 10 launches of 4.8 that added the ranges up into a buffer of their own).
constexpr int ADAM_MEM = 16;
struct AdamBias { float c1[ADAM_MEM], c2[ADAM_MEM]; };   // bias corrections of members mem0 .. of this launch
__global__ void k_adam(float* p, float* gr, const float* part, int S, long long sRange, float* m1, float* m2, bf16* pb,
                       bf16* pbf, bf16* pbt, FragMap map, long long P, int mem0, AdamBias bias, float lr, float b1, float b2,
                       float eps) {
  const long long o = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= P) return;
  const int q = blockIdx.y;
  const long long e = (long long)(mem0 + q) * P + o;
  float g;
  if (S > 1) {
    g = 0.0f;
    for (int s = 0; s < S; ++s) g += part[s * sRange + e];
    gr[e] = g;
  } else {
    g = gr[e];
  }
  const float a = b1 * m1[e] + (1.0f - b1) * g;
  const float b = b2 * m2[e] + (1.0f - b2) * g * g;
  m1[e] = a;
  m2[e] = b;
  const float mh = a / bias.c1[q], vh = b / bias.c2[q];
  const float w = p[e] - lr * mh / (sqrtf(vh) + eps);
  p[e] = w;
  store_bf16(pb, pbf, pbt, map, (long long)(mem0 + q) * P, o, w);
}

// ensemble mean and population variance of the de-normalised outputs (and per-member outputs)
__global__ void k_ensemble(const float* out, long long sOut, int ldo, int K, int B, int dout, const float* ymu,
                           const float* ysd, float* mean, float* var, float* members) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (long long)B * dout) return;
  const int m = (int)(e / dout), n = (int)(e % dout);
  float s = 0.0f;
  for (int k = 0; k < K; ++k) {
    const float y = out[k * sOut + (long long)m * ldo + n] * ysd[n] + ymu[n];
    if (members) members[(long long)k * B * dout + e] = y;
    s += y;
  }
  const float mu = s / (float)K;
  if (mean) mean[e] = mu;
  if (var) {
    float q = 0.0f;
    for (int k = 0; k < K; ++k) {
      const float d = out[k * sOut + (long long)m * ldo + n] * ysd[n] + ymu[n] - mu;
      q += d * d;
    }
    var[e] = q / (float)K;
  }
}

// per-column mean and population standard deviation of n rows (one block per column)
constexpr int FIT_NT = 256;
__global__ __launch_bounds__(FIT_NT) void k_fit_norm(const float* X, int n, int d, float* mu, float* sd) {
  __shared__ double sh[FIT_NT];
  const int c = blockIdx.x;
  double s = 0.0;
  for (int r = threadIdx.x; r < n; r += FIT_NT) s += X[(long long)r * d + c];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = FIT_NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  const double m = sh[0] / n;
  __syncthreads();
  s = 0.0;
  for (int r = threadIdx.x; r < n; r += FIT_NT) {
    const double q = X[(long long)r * d + c] - m;
    s += q * q;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = FIT_NT / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    mu[c] = (float)m;
    sd[c] = (float)fmax(sqrt(sh[0] / n), 1e-6);
  }
}

}  // namespace rsur
