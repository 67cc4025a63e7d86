// af_learn.hip -- the learned blend coefficient of the 2D cell-average fluxes
// on gfx950: face features, inference of the 40-64-64-1 network on the MFMA
// units, and the network's training (loss gradient and Adam).
//
// The network proposes, per face, the coefficient that blends the low- and
// high-order cell-average fluxes in place of the smoothness blend theta^s of
// Sec. 3.2; the density/pressure limiter of Sec. 3.3 then clamps it as it
// clamps theta^s (the coefficient used is theta_nn theta^rho theta^p, never
// above theta_nn nor the admissible bound), and the face flux stays
// single-valued (conservative).
//
// Features of a face (a, b its minus and plus cells): in the face's frame
// (normal n along its axis, tangent t along the other) the 4 x 3 block of
// cell averages at normal offsets -2, -1 (a), +1 (b), +2 and tangential
// offsets -1, 0, +1, ghost cells being boundary images.  With face values
// rho_f = (rho_a + rho_b)/2, p_f, u_nf, u_tf likewise and
// c_f = sqrt(gamma p_f / rho_f): for s = -1, 0, +1 and m = -2, -1, +1, +2 the
// triple [ln(p / p_f), (u_n - u_nf) / c_f, (u_t - u_tf) / c_f], then
// ln(rho / rho_f) for m = -2, -1, +1, +2 at s = 0 (40 values).
//
// Network: h1 = tanh(W1 x + b1), h2 = tanh(W2 h1 + b2), z = w3.h2 + b3,
// theta_nn = min(max(z, 0), 1); parameters as one FP32 vector
// [W1 (64 x 40, row-major), b1, W2 (64 x 64), b2, w3, b3].  Inference keeps
// W1, W2, w3 and the layer inputs x, h1 in bfloat16 (round to nearest even)
// and accumulates in FP32 (MFMA 32x32x16 bf16); training runs in FP32.
#include "af_device.hpp"
#include "af_internal.hpp"
#include "af_lattice.hpp"

using namespace afd;

namespace {

constexpr int NIN = afi::kMlpIn, NH = afi::kMlpHidden;
constexpr int OFF_W1 = 0, OFF_B1 = NH * NIN, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH;
static_assert(OFF_B3 + 1 == afi::kMlpParams, "parameter layout");

// two values rounded to nearest even, the first in the low half (one hardware
// conversion on gfx950)
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 v = {(__bf16)x, (__bf16)y};
  return __builtin_bit_cast(unsigned, v);
}
// (rho, u, v, p) as FP32 from a cell average (FP64 arithmetic)
__device__ __forceinline__ void prims_of(double gm1, const double* V, float* P) {
  const double ir = 1.0 / V[0], u = V[1] * ir, v = V[2] * ir;
  P[0] = float(V[0]);
  P[1] = float(u);
  P[2] = float(v);
  P[3] = float(gm1 * (V[3] - 0.5 * V[0] * (u * u + v * v)));
}

__device__ __forceinline__ float pos_or_tiny(float v) { return v > 1e-30f ? v : 1e-30f; }

// ln(x) from the hardware's log2, for x > 0 (values below the normal ones count
// as the smallest of those)
__device__ __forceinline__ float ln_fast(float x) {
  // ln 2 in two parts, so that the product rounds once
  constexpr float hi = 0.693147182464599609375f, lo = -1.90465429995776787854e-9f;
  const float l = __builtin_amdgcn_logf(fmaxf(x, 0x1p-126f));
  const float r = l * hi;
  return r + fmaf(l, lo, fmaf(l, hi, -r));
}

// half H of the features of a face from the primitives of its stencil cells:
// cell(s, q, P) fills (rho, u_n, u_t, p) in the face's frame of tangential
// offset s-1 and normal offset q in (-2, -1, +1, +2).  The half is the triples
// of stencil cells 6H .. 6H+5 (cell 4s+q), features 18H .. 18H+17, and the
// density ratios of q = 2H, 2H+1, features 36+2H, 37+2H: twenty values f.
template <int H, typename CellFn>
__device__ __forceinline__ void features_of(float gam, CellFn cell, float* f) {
  // face values from the two cells that adjoin the face
  float A[4], B[4];
  cell(1, 1, A);
  cell(1, 2, B);
  const float rf = 0.5f * (A[0] + B[0]), pf = 0.5f * (A[3] + B[3]);
  const float unf = 0.5f * (A[1] + B[1]), utf = 0.5f * (A[2] + B[2]);
  const float pt = pos_or_tiny(pf), rt = pos_or_tiny(rf);
  const float ipf = rcp(pt), irf = rcp(rt);
  // gamma p / rho: the quotient by the reciprocal, rounded as the division
  const float gp = gam * pt;
  float c2 = gp * irf;
  c2 = fmaf(fmaf(-rt, c2, gp), irf, c2);
  const float icf = rcp(root(c2));
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    float P[4];
    cell((6 * H + c) / 4, (6 * H + c) % 4, P);
    f[3 * c] = ln_fast(pos_or_tiny(P[3]) * ipf);
    f[3 * c + 1] = (P[1] - unf) * icf;
    f[3 * c + 2] = (P[2] - utf) * icf;
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    float P[4];
    cell(1, 2 * H + q, P);
    f[18 + q] = ln_fast(pos_or_tiny(P[0]) * irf);
  }
}

// 1 / (1 + e^{2x}) with the hardware exponential and reciprocal: tanh x is
// 1 - 2 of it (the result feeds bfloat16 operands; its error is far below their
// rounding)
__device__ __forceinline__ float sigma_fast(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * 2.885390043258666992f));
}
__device__ __forceinline__ float tanh_fast(float x) { return 1.0f - 2.0f * sigma_fast(x); }

// ---------------------------------------------------------------------------
// Blocks of faces: a workgroup of 256 threads takes up to 128 consecutive
// faces of each of up to eight rows of one direction and holds the primitives
// of their stencil cells in LDS (ten rows of cells for eight rows of x-faces,
// eleven for y-faces, where one face row at a time needed three or four).
// ---------------------------------------------------------------------------
constexpr int IB = 128;                 // faces per row of a block
constexpr int RB = 8;                   // face rows per block, at most
constexpr int CW = IB + 4;              // stencil cells per row
typedef float CellBlock[4][RB + 3][CW]; // [component][row][column]

// how the faces of a grid are cut into blocks of rb rows
struct FaceBlocks {
  int nsegx, nsegy, rb;
  long nbx, nblocks;  // blocks of x-faces, all blocks
};

// block blk: direction, first row and row count, first face along the
// rows, face count per row, and its stencil cells: x-faces need columns
// i0-2 .. i0+cnt and rows row0-1 .. row0+nr, y-faces columns i0-1 ..
// i0+cnt and rows row0-2 .. row0+nr-1
struct FaceBlock {
  int d, row0, nr, i0, cnt, ncol, nrow, c0, r0;
};
__device__ __forceinline__ FaceBlock block_of(const G2& g, const FaceBlocks& fb, long blk) {
  FaceBlock b;
  if (blk < fb.nbx) {
    b.d = 0;
    b.row0 = (int)(blk / fb.nsegx) * fb.rb;
    b.nr = min(fb.rb, g.n2 - b.row0);
    b.i0 = (int)(blk % fb.nsegx) * IB;
    b.cnt = min(IB, g.n1 + 1 - b.i0);
  } else {
    b.d = 1;
    const long r = blk - fb.nbx;
    b.row0 = (int)(r / fb.nsegy) * fb.rb;
    b.nr = min(fb.rb, g.n2 + 1 - b.row0);
    b.i0 = (int)(r % fb.nsegy) * IB;
    b.cnt = min(IB, g.n1 - b.i0);
  }
  b.ncol = b.d == 0 ? b.cnt + 3 : b.cnt + 2;
  b.nrow = (b.d == 0 ? 2 : 3) + b.nr;
  b.c0 = b.d == 0 ? b.i0 - 2 : b.i0 - 1;
  b.r0 = b.d == 0 ? b.row0 - 1 : b.row0 - 2;
  return b;
}

// the primitives of block b's stencil cells into LDS, by all 256 threads: the
// loads of the FP64 averages are all issued, then a barrier (the previous
// block's readers are done), then the stores
__device__ __forceinline__ void stage_cells(const G2& g, double gm1, const double* __restrict__ U,
                                            const FaceBlock& b, CellBlock& cell) {
  constexpr int CPT = ((RB + 3) * (IB + 2) + 255) / 256;
  static_assert((RB + 2) * (IB + 3) <= CPT * 256 && (RB + 3) * (IB + 2) <= CPT * 256,
                "cells per thread");
  const int tid = threadIdx.x;
  double pre[CPT][4];
#pragma unroll
  for (int r = 0; r < CPT; ++r) {
    const int e = tid + 256 * r;
    if (e < b.ncol * b.nrow)
      raw_value(g, U, 2 * (b.c0 + e % b.ncol) + 1, 2 * (b.r0 + e / b.ncol) + 1, pre[r]);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < CPT; ++r) {
    const int e = tid + 256 * r;
    if (e < b.ncol * b.nrow) {
      float P[4];
      prims_of(gm1, pre[r], P);
#pragma unroll
      for (int k = 0; k < 4; ++k) cell[k][e / b.ncol][e % b.ncol] = P[k];
    }
  }
}

// half h of the features of face (i0 + fl, row) of block b; direction and half
// are the same for a wave, and known to the code that reads the cells, so that
// all reads of a face share one address
template <int D, int H>
__device__ __forceinline__ void face_features(const FaceBlock& b, const CellBlock& cell, float gam,
                                              int fl, int row, float* f) {
  // the cell of the face's own index, the one on its plus side
  const float* at = &cell[0][row - b.r0][b.i0 + fl - b.c0];
  constexpr int plane = (RB + 3) * CW;
  features_of<H>(gam,
                 [&](int s, int q, float* P) {
                   const float* c = at + (D == 0 ? (s - 1) * CW + q - 2 : (q - 2) * CW + s - 1);
                   P[0] = c[0];
                   P[1] = c[(1 + D) * plane];
                   P[2] = c[(2 - D) * plane];
                   P[3] = c[3 * plane];
                 },
                 f);
}
__device__ __forceinline__ void block_features(const FaceBlock& b, const CellBlock& cell, float gam,
                                               int fl, int row, int h, float* f) {
  if (b.d == 0) {
    if (h == 0)
      face_features<0, 0>(b, cell, gam, fl, row, f);
    else
      face_features<0, 1>(b, cell, gam, fl, row, f);
  } else {
    if (h == 0)
      face_features<1, 0>(b, cell, gam, fl, row, f);
    else
      face_features<1, 1>(b, cell, gam, fl, row, f);
  }
}

// index of the first face of a block's row
__device__ __forceinline__ long first_face(const G2& g, const FaceBlock& b, int row) {
  return b.d == 0 ? (long)row * (g.n1 + 1) + b.i0
                  : (long)g.n2 * (g.n1 + 1) + (long)row * g.n1 + b.i0;
}

// ---------------------------------------------------------------------------
// features of every face (training data).  The output, 160 bytes a face, is
// what the kernel has to move: two threads form a face's features, a row of
// 128 faces passes through LDS and is written as one contiguous run.  (One
// thread per face with its own 40 stores, 160 bytes apart between lanes, and
// its 18 cells' primitives formed again for every face, took 64 us at
// 500 x 250, 0.7 TB/s; the copy rate is 5.1 TB/s.)
// ---------------------------------------------------------------------------
constexpr int OROW = NIN + 1;  // LDS row (floats): lanes 41 apart fall on different banks

__global__ void __launch_bounds__(256) k_features(G2 g, double gm1, float gam,
                                                  const double* __restrict__ U,
                                                  float* __restrict__ out, FaceBlocks fb) {
  __shared__ CellBlock cell;
  __shared__ float feat[IB * OROW];
  const int tid = threadIdx.x, fl = tid & (IB - 1);
  const int half = __builtin_amdgcn_readfirstlane(tid / IB);
  for (long blk = blockIdx.x; blk < fb.nblocks; blk += gridDim.x) {
    const FaceBlock B = block_of(g, fb, blk);
    stage_cells(g, gm1, U, B, cell);
    for (int rr = 0; rr < B.nr; ++rr) {
      const int row = B.row0 + rr;
      __syncthreads();  // the cells are in; the previous row is written
      if (fl < B.cnt) {
        float f[20];
        block_features(B, cell, gam, fl, row, half, f);
        float* o = feat + fl * OROW;
#pragma unroll
        for (int n = 0; n < 18; ++n) o[18 * half + n] = f[n];
        o[36 + 2 * half] = f[18];
        o[37 + 2 * half] = f[19];
      }
      __syncthreads();
      float* o = out + first_face(g, B, row) * NIN;
      for (int e = tid; e < B.cnt * NIN; e += 256) o[e] = feat[e / NIN * OROW + e % NIN];
    }
  }
}

// ---------------------------------------------------------------------------
// inference.  For each face row of a block (above) the four wave64s of a
// workgroup write the features as bfloat16 rows; each wave
// then runs the network on 32 faces with MFMA 32x32x16 bf16 in the
// transposed form H^T = W X^T: the weights are the A operand (units x
// inputs, in registers), the faces the columns.  A 32 x 32 accumulator holds
// in lane (face c, half h) the rows (units) 8 (r/4) + 4 h + r%4 of column c,
// r = 0..15, and the B operand of the next layer needs in that lane the
// inputs 16 kb + 8 h + e, e = 0..7, of the same face: registers 8q .. 8q+7
// of the accumulator of unit block nb are exactly that for kb = 2 nb + q,
// once the hidden units are numbered in that (virtual) order, which is how
// layer 2's weights are stored.  So hidden values never leave the
// registers, and the output layer's sum over units ends with one exchange
// between the two halves of the wave.
//
// The vector units bound it: 128 activations of an exponential and a
// reciprocal per face, then the features.  Activations of six instructions
// (output layer: four) and features that share an address, one reciprocal per
// quotient and packed stores take 62 us at 1000 x 500 and 237 at 2048 x 1024
// (eight and six, and features selected by direction and half: 74 and 277).
// ---------------------------------------------------------------------------
constexpr int KIN = 48;                 // inputs padded to three K steps of 16
constexpr int FROW = KIN + 8;           // feature row (bf16; 16-byte aligned)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct InferShared {
  CellBlock cell;
  unsigned short feat[IB * FROW];
  float b1[NH], b2[NH], w3[NH];         // biases, and -2 times the output weights (bf16 values)
  // layer 2's A operands, per lane (in LDS rather than registers: with them
  // in registers the kernel holds 188 VGPRs, two waves per SIMD, and ran 18 %
  // slower at 2048 x 1024)
  bf16x8 a2[2][4][64];
};

// four floats, which need no more than a float's alignment
__device__ __forceinline__ f32x4 load4(const float* p) {
  f32x4 v;
  __builtin_memcpy(&v, p, sizeof(v));
  return v;
}

// unit of layer-2 input (virtual) index k, for the half h of the lanes that
// holds it: kb = k / 16 = 2 nb + q, e = k % 8 = 4 a + i (see above)
__device__ __forceinline__ int hidden_unit(int kb, int h, int e) {
  const int nb = kb >> 1, q = kb & 1, a = e >> 2, i = e & 3;
  return 32 * nb + 8 * (2 * q + a) + 4 * h + i;
}

// at least three waves per SIMD (at most 168 VGPRs)
__global__ void __launch_bounds__(256, 3) k_infer(G2 g, double gm1, float gam,
                                               const double* __restrict__ U,
                                               const float* __restrict__ p,
                                               float* __restrict__ theta, FaceBlocks fb) {
  __shared__ InferShared S;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int h = lane >> 5, c32 = lane & 31;
  // A operands: lane (m = c32, h) holds row 32 nb + m, inputs 16 kb + 8 h + e
  // (layer 2's written to LDS by the first wave, read after the first
  // barrier), from the FP32 parameters: each workgroup rounds them for itself
  // (27 KB from L2), which spares a packing launch of 4.7 us per inference
  bf16x8 A1[2][3];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
    for (int kb = 0; kb < 3; ++kb) {
      const int k0 = 16 * kb + 8 * h;  // 40: past the inputs
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const f32x4 x = load4(p + OFF_W1 + (32 * nb + c32) * NIN + (k0 < NIN ? k0 : 0) + 4 * a);
#pragma unroll
        for (int i = 0; i < 4; ++i) A1[nb][kb][4 * a + i] = (__bf16)(k0 < NIN ? x[i] : 0.0f);
      }
    }
    if (wave == 0) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        bf16x8 v;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          // four consecutive units (see hidden_unit)
          const f32x4 x = load4(p + OFF_W2 + (32 * nb + c32) * NH + hidden_unit(kb, h, 4 * a));
#pragma unroll
          for (int i = 0; i < 4; ++i) v[4 * a + i] = (__bf16)x[i];
        }
        S.a2[nb][kb][lane] = v;
      }
    }
  }
  static_assert(NIN % 8 == 0, "whole groups of eight inputs");
  if (tid < IB)  // inputs 40..47 of every face are zero
#pragma unroll
    for (int n = 0; n < KIN - NIN; ++n) S.feat[tid * FROW + NIN + n] = 0;
  if (tid < NH) {
    S.b1[tid] = p[OFF_B1 + tid];
    S.b2[tid] = p[OFF_B2 + tid];
    S.w3[tid] = -2.0f * (float)(__bf16)p[OFF_W3 + tid];
  }
  float z0 = p[OFF_B3];  // plus the sum of the output weights: z where all sigma are 0
#pragma unroll 8
  for (int k = 0; k < NH; ++k) z0 += (float)(__bf16)p[OFF_W3 + k];
  for (long blk = blockIdx.x; blk < fb.nblocks; blk += gridDim.x) {
    // (held one block ahead, the loads of the averages took more registers
    // than three workgroups per CU leave; the other workgroups on the CU hide
    // the wait)
    const FaceBlock B = block_of(g, fb, blk);
    stage_cells(g, gm1, U, B, S.cell);
    const int cnt = B.cnt;
    for (int rr = 0; rr < B.nr; ++rr) {
      const int row = B.row0 + rr;
      __syncthreads();  // the cells are in; the previous row is done with the features
      {
        // two threads per face, one half of its features each
        const int fl = tid & (IB - 1), half = __builtin_amdgcn_readfirstlane(tid / IB);
        float f[20];
#pragma unroll
        for (int n = 0; n < 20; ++n) f[n] = 0.0f;
        if (fl < cnt) block_features(B, S.cell, gam, fl, row, half, f);
        unsigned* fo = reinterpret_cast<unsigned*>(S.feat + fl * FROW);
#pragma unroll
        for (int n = 0; n < 9; ++n) fo[9 * half + n] = pack_bf16(f[2 * n], f[2 * n + 1]);
        fo[18 + half] = pack_bf16(f[18], f[19]);
      }
      __syncthreads();
      // the wave's 32 faces: lane (c32, h) works on face 32 wave + c32
      const unsigned short* fa = S.feat + (32 * wave + c32) * FROW;
      f32x16 acc[2];
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nb][r] = 0.0f;
#pragma unroll
      for (int kb = 0; kb < 3; ++kb) {
        const bf16x8 x = *reinterpret_cast<const bf16x8*>(fa + 16 * kb + 8 * h);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1[nb][kb], x, acc[nb], 0, 0, 0);
      }
      // h1 = tanh(W1 x + b1) in bfloat16: layer 2's B operand, kb = 2 nb + q
      bf16x8 hb[4];
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 bias = *reinterpret_cast<const float4*>(&S.b1[32 * nb + 8 * j + 4 * h]);
          const float bj[4] = {bias.x, bias.y, bias.z, bias.w};
#pragma unroll
          for (int i = 0; i < 4; ++i)
            hb[2 * nb + (j >> 1)][4 * (j & 1) + i] = (__bf16)tanh_fast(acc[nb][4 * j + i] + bj[i]);
        }
      // layer 2, summed up from its bias
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 bias = *reinterpret_cast<const float4*>(&S.b2[32 * nb + 8 * j + 4 * h]);
          acc[nb][4 * j] = bias.x;
          acc[nb][4 * j + 1] = bias.y;
          acc[nb][4 * j + 2] = bias.z;
          acc[nb][4 * j + 3] = bias.w;
        }
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(S.a2[nb][kb][lane], hb[kb], acc[nb], 0, 0, 0);
      // z = w3 . tanh(W2 h1 + b2) + b3, as (sum of w3 + b3) + (-2 w3) . sigma:
      // this lane's 32 units of its face, then the other half's 32 from the
      // lane 32 away
      float z = 0.0f;
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float4 ow = *reinterpret_cast<const float4*>(&S.w3[32 * nb + 8 * j + 4 * h]);
          z += ow.x * sigma_fast(acc[nb][4 * j]);
          z += ow.y * sigma_fast(acc[nb][4 * j + 1]);
          z += ow.z * sigma_fast(acc[nb][4 * j + 2]);
          z += ow.w * sigma_fast(acc[nb][4 * j + 3]);
        }
      z += __shfl_xor(z, 32, 64);
      const int m = 32 * wave + c32;
      if (h == 0 && m < cnt) {
        const long f = first_face(g, B, row) + m;
        theta[f] = fminf(fmaxf(z + z0, 0.0f), 1.0f);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// training: gradient of the mean squared error over n samples, FP32.  A
// workgroup (four wave64s) takes chunks of 16 samples through the forward
// and backward pass with MFMA 16x16x4 FP32 (FP32 products and sums, as the
// vector units form them): wave w owns hidden units 16w .. 16w+15 of every
// layer, its slices of W1, W2 and W2^T stay in registers, and only the
// activations and their derivatives pass through LDS.  Its share of the
// gradient accumulates in registers; partial gradients are summed in a fixed
// order (deterministic).
//
// What bounds a minibatch of 1024 rows is latency, not arithmetic (41 MFLOP,
// 0.3 us at the matrix rate): hence chunks of the smallest matrix tile, 64
// workgroups, and 70 matrix instructions in a row per wave (1 us).  Chunks of
// 64 samples on the vector units, with weight rows read from LDS 64 banks
// apart by the lanes of a wave, took 194 us per minibatch.
// ---------------------------------------------------------------------------
constexpr int GC = 16;             // samples per chunk
constexpr int GT = 256;            // threads per workgroup
constexpr int kGradBlocks = 256;   // partial gradients at most
// LDS rows: sample rows of 68 (activations) and 44 (inputs) floats put the 16
// rows x 4 columns a matrix operand reads into 64 different banks
constexpr int HS = NH + 4, XS = NIN + 4;

struct GradShared {
  float X[GC * XS], H1[GC * HS], A2[GC * HS], A1[GC * HS], zp[4][GC], y[GC];
};

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// sum over the 16 lanes of each quarter of a wave
__device__ __forceinline__ float sum16(float v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// sum over the four quarters of a wave
__device__ __forceinline__ float sum_quarters(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

__global__ void __launch_bounds__(GT) k_grad(const float* __restrict__ X,
                                             const float* __restrict__ y, long n,
                                             const float* __restrict__ p,
                                             float* __restrict__ part, float inv_n) {
  __shared__ GradShared S;
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  // operand coordinates of the lane: A[c][q], B[q][c], D[4 q + r][c]
  const int c = lane & 15, q = lane >> 4;
  const int u = 16 * w + c;  // this lane's unit (column) in every layer
  // B operands: W1^T and W2^T (forward) and W2 (backward), column u
  float bW1[NIN / 4], bW2[NH / 4], bW2t[NH / 4];
#pragma unroll
  for (int s = 0; s < NIN / 4; ++s) bW1[s] = p[OFF_W1 + u * NIN + 4 * s + q];
#pragma unroll
  for (int s = 0; s < NH / 4; ++s) {
    bW2[s] = p[OFF_W2 + u * NH + 4 * s + q];
    bW2t[s] = p[OFF_W2 + (4 * s + q) * NH + u];
  }
  const float b1 = p[OFF_B1 + u], b2 = p[OFF_B2 + u], w3 = p[OFF_W3 + u], b3 = p[OFF_B3];
  f32x4 gW2[4], gW1[3];
#pragma unroll
  for (int k = 0; k < 4; ++k) gW2[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 3; ++k) gW1[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gb1 = 0.f, gb2 = 0.f, gw3 = 0.f, gb3 = 0.f, loss = 0.f;
  const long nchunk = (n + GC - 1) / GC;
  for (long ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
    const long base = ch * GC;
    __syncthreads();  // the previous chunk is done with the LDS
    for (int e = t; e < GC * XS; e += GT) {
      const long row = base + e / XS;
      S.X[e] = (row < n && e % XS < NIN) ? X[row * NIN + e % XS] : 0.f;
    }
    if (t < GC) S.y[t] = base + t < n ? y[base + t] : 0.f;
    __syncthreads();
    // layer 1: H1 = tanh(X W1^T + b1)
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NIN / 4; ++s) acc = mfma4(S.X[c * XS + 4 * s + q], bW1[s], acc);
    float h1[4], h2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h1[r] = tanhf(acc[r] + b1);
      S.H1[(4 * q + r) * HS + u] = h1[r];
    }
    __syncthreads();
    // layer 2, and this wave's units' share of z = w3 . H2 + b3
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NH / 4; ++s) acc = mfma4(S.H1[c * HS + 4 * s + q], bW2[s], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h2[r] = tanhf(acc[r] + b2);
      const float zs = sum16(w3 * h2[r]);
      if (c == 0) S.zp[w][4 * q + r] = zs;
    }
    __syncthreads();
    // residuals, dL/d(layer-2 pre-activation)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 4 * q + r;
      const float z = ((S.zp[0][m] + S.zp[1][m]) + (S.zp[2][m] + S.zp[3][m])) + b3;
      const float res = base + m < n ? z - S.y[m] : 0.f;
      const float dz = 2.f * res * inv_n;
      const float a2 = dz * w3 * (1.f - h2[r] * h2[r]);
      gw3 += dz * h2[r];
      gb2 += a2;
      gb3 += dz;
      loss += res * res;
      S.A2[m * HS + u] = a2;
    }
    __syncthreads();
    // dL/d(layer-1 pre-activation) = (A2 W2) (1 - H1^2)
    acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NH / 4; ++s) acc = mfma4(S.A2[c * HS + 4 * s + q], bW2t[s], acc);
    // gradient of W2, rows 16w .. 16w+15: A2^T H1 over the samples
#pragma unroll
    for (int s = 0; s < GC / 4; ++s) {
      const float a = S.A2[(4 * s + q) * HS + u];
#pragma unroll
      for (int k = 0; k < 4; ++k) gW2[k] = mfma4(a, S.H1[(4 * s + q) * HS + 16 * k + c], gW2[k]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float a1 = acc[r] * (1.f - h1[r] * h1[r]);
      gb1 += a1;
      S.A1[(4 * q + r) * HS + u] = a1;
    }
    // gradient of W1, rows 16w ..: A1^T X; only this wave's own columns of
    // A1 are read, so its own LDS order suffices, but the compiler is told
    __syncthreads();
#pragma unroll
    for (int s = 0; s < GC / 4; ++s) {
      const float a = S.A1[(4 * s + q) * HS + u];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int col = 16 * k + c;
        const float x = S.X[(4 * s + q) * XS + (col < XS ? col : XS - 1)];  // columns 40.. are 0
        gW1[k] = mfma4(a, x, gW1[k]);
      }
    }
  }
  // this workgroup's partial gradient and loss sum
  float* o = part + (long)blockIdx.x * (afi::kMlpParams + 1);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 16 * w + 4 * q + r;
#pragma unroll
    for (int k = 0; k < 4; ++k) o[OFF_W2 + row * NH + 16 * k + c] = gW2[k][r];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (16 * k + c < NIN) o[OFF_W1 + row * NIN + 16 * k + c] = gW1[k][r];
  }
  gb1 = sum_quarters(gb1);
  gb2 = sum_quarters(gb2);
  gw3 = sum_quarters(gw3);
  gb3 = sum_quarters(gb3);  // the same sum in every lane of every wave
  loss = sum_quarters(loss);
  if (q == 0) {
    o[OFF_B1 + u] = gb1;
    o[OFF_B2 + u] = gb2;
    o[OFF_W3 + u] = gw3;
  }
  if (t == 0) {
    o[OFF_B3] = gb3;
    o[afi::kMlpParams] = loss;
  }
}

// one Adam update of parameter e
__device__ __forceinline__ void adam_one(float* p, float ge, float* m, float* v, int e, float lr,
                                         float c1, float c2) {
  const float me = 0.9f * m[e] + 0.1f * ge;
  const float ve = 0.999f * v[e] + 0.001f * ge * ge;
  m[e] = me;
  v[e] = ve;
  p[e] -= lr * (me * c1) / (sqrtf(ve * c2) + 1e-8f);
}

// Sum of the partial gradients, and (ADAM) the update that uses it: 64
// elements a workgroup, a quarter of the partials per wave (one thread per
// element over all 16 partials of a minibatch of 1024 took 5.3 us, and the
// update another launch of 4.7 us)
template <bool ADAM>
__global__ void __launch_bounds__(256) k_grad_sum(const float* __restrict__ part, int nparts,
                                                  float* __restrict__ grad,
                                                  float* __restrict__ loss, float inv_n,
                                                  float* __restrict__ p, float* __restrict__ m,
                                                  float* __restrict__ v, float lr, float c1,
                                                  float c2) {
  __shared__ float sh[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const int b0 = w * nparts / 4, b1 = (w + 1) * nparts / 4;
  float s = 0.f;
  if (e <= afi::kMlpParams) {
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += part[(long)b * (afi::kMlpParams + 1) + e];
  }
  sh[w][lane] = s;
  __syncthreads();
  if (w != 0 || e > afi::kMlpParams) return;
  s = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
  if (e == afi::kMlpParams) {
    if (loss) *loss = s * inv_n;
    return;
  }
  grad[e] = s;
  if constexpr (ADAM) adam_one(p, s, m, v, e, lr, c1, c2);
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float lr, float c1, float c2) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < afi::kMlpParams) adam_one(p, g[e], m, v, e, lr, c1, c2);
}

}  // namespace

namespace afi {

// persistent workgroups of kernel K (256 threads): as many as are resident
template <typename K>
static int resident(K kernel, int (&cache)[64]) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (cache[dev] == 0) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, 256, 0) != hipSuccess ||
        per <= 0)
      per = 1;
    cache[dev] = cus * per;
  }
  return cache[dev];
}

// the blocks of a grid's faces for nwg workgroups.  Rows per block: the most
// (up to RB) that still leave every resident workgroup two blocks, so that a
// small grid keeps the device busy
static FaceBlocks face_blocks(const G2& g, long nwg) {
  FaceBlocks fb;
  fb.nsegx = (g.n1 + 1 + IB - 1) / IB;
  fb.nsegy = (g.n1 + IB - 1) / IB;
  auto bx = [&](int rb) { return (long)((g.n2 + rb - 1) / rb) * fb.nsegx; };
  auto all = [&](int rb) { return bx(rb) + (long)((g.n2 + 1 + rb - 1) / rb) * fb.nsegy; };
  fb.rb = RB;
  while (fb.rb > 1 && all(fb.rb) < 2 * nwg) fb.rb /= 2;
  fb.nbx = bx(fb.rb);
  fb.nblocks = all(fb.rb);
  return fb;
}

hipError_t blend_features(const Geo& geo, const Phys& ph, const double* U, float* feat,
                          hipStream_t s) {
  static int cache[64] = {0};
  const G2 g = stage_geo(geo);
  const long nwg = resident(k_features, cache);
  const FaceBlocks fb = face_blocks(g, nwg);
  hipLaunchKernelGGL(k_features, dim3((unsigned)(fb.nblocks < nwg ? fb.nblocks : nwg)), dim3(256),
                     0, s, g, ph.gm1, float(ph.gam), U, feat, fb);
  return hipGetLastError();
}

hipError_t blend_infer(const Geo& geo, const Phys& ph, const double* U, const float* params,
                       float* theta, hipStream_t s, Timer* tm) {
  static int cache[64] = {0};
  const G2 g = stage_geo(geo);
  const long nwg = resident(k_infer, cache);
  const FaceBlocks fb = face_blocks(g, nwg);
  AFI_TIMED(tm, 8, s,
            hipLaunchKernelGGL(k_infer, dim3((unsigned)(fb.nblocks < nwg ? fb.nblocks : nwg)),
                               dim3(256), 0, s, g, ph.gm1, float(ph.gam), U,
                               params, theta, fb));
  return hipGetLastError();
}

size_t mlp_grad_workspace(long n) {
  (void)n;
  return sizeof(float) * (size_t)kGradBlocks * (kMlpParams + 1);
}

// bias corrections of Adam's moments after `step` updates
static void adam_coefs(long step, float& c1, float& c2) {
  c1 = float(1.0 / (1.0 - pow(0.9, (double)step)));
  c2 = float(1.0 / (1.0 - pow(0.999, (double)step)));
}

// the partial gradients of the n rows; returns their number
static int grad_parts(const float* X, const float* y, long n, const float* params, float* part,
                      hipStream_t s) {
  const long nchunk = (n + GC - 1) / GC;
  const int nb = (int)(nchunk < kGradBlocks ? nchunk : kGradBlocks);
  hipLaunchKernelGGL(k_grad, dim3(nb), dim3(GT), 0, s, X, y, n, params, part, 1.0f / float(n));
  return nb;
}

constexpr int kSumBlocks = (int)((kMlpParams + 1 + 63) / 64);

hipError_t mlp_grad(const float* X, const float* y, long n, const float* params, float* grad,
                    float* loss, void* ws, hipStream_t s) {
  float* part = (float*)ws;
  const int nb = grad_parts(X, y, n, params, part, s);
  hipLaunchKernelGGL((k_grad_sum<false>), dim3(kSumBlocks), dim3(256), 0, s, (const float*)part,
                     nb, grad, loss, 1.0f / float(n), (float*)nullptr, (float*)nullptr,
                     (float*)nullptr, 0.f, 0.f, 0.f);
  return hipGetLastError();
}

hipError_t mlp_step(const float* X, const float* y, long n, float* params, float* grad, float* m,
                    float* v, long step, float lr, float* loss, void* ws, hipStream_t s) {
  float* part = (float*)ws;
  const int nb = grad_parts(X, y, n, params, part, s);
  float c1, c2;
  adam_coefs(step, c1, c2);
  hipLaunchKernelGGL((k_grad_sum<true>), dim3(kSumBlocks), dim3(256), 0, s, (const float*)part, nb,
                     grad, loss, 1.0f / float(n), params, m, v, lr, c1, c2);
  return hipGetLastError();
}

hipError_t mlp_adam(float* params, const float* grad, float* m, float* v, long step, float lr,
                    hipStream_t s) {
  float c1, c2;
  adam_coefs(step, c1, c2);
  hipLaunchKernelGGL(k_adam, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, params, grad, m, v,
                     lr, c1, c2);
  return hipGetLastError();
}

}  // namespace afi
