// Parameter packing, and the hand-written backward pass of the VMC gradient
// (Sec. 3, Eq. grad): the sample forward is recomputed per chunk of samples
// (activations of connected configurations are never stored), the output
// seeds are built from the local energies, and masked GEMMs propagate them to
// every weight and bias.
#include <algorithm>

#include "nqs_internal.h"

namespace nqs {

// ------------------------------------------------------------------ masks
// In original (unpacked) indexing; degrees: qubit j -> 1 + pos[j], hidden
// unit k -> 1 + k mod (n-1).
enum MaskKind { MK_NONE = 0, MK_L1 = 1, MK_HID = 2, MK_HEAD_O = 3, MK_HEAD_P = 4 };

__device__ __forceinline__ bool mask_at(const Geom& g, int kind, int row, int col) {
  const int nm1 = g.n - 1;
  switch (kind) {
    case MK_L1: return (row % nm1) + 1 >= g.pos[col] + 1;
    case MK_HID: return (row % nm1) >= (col % nm1);
    case MK_HEAD_O: return g.pos[row] + 1 > (col % nm1) + 1;
    case MK_HEAD_P: return (col % nm1) + 1 <= g.n - 2;
  }
  return true;
}

// Which tensor of the flat layout holds parameter p: returns kind and
// (row, col) for weights, or -1 kind for a bias.  The layers of a separate
// phase network and its head are dense (MK_NONE).
__device__ __forceinline__ void locate(const Geom& g, long long p, int& tensor, int& kind, int& row,
                                       int& col, int& in) {
  const int L = g.L;
  const int ntens = g.phase_mode ? 4 * L + 4 : 2 * L + 4;
  int t = 0;
  while (t + 1 < ntens && p >= g.poff[t + 1]) ++t;
  tensor = t;
  const long long local = p - g.poff[t];
  if (g.phase_mode && t >= 2 * L + 2 && t < 4 * L + 2) {
    const int l = (t - 2 * L - 2) / 2 + 1;
    in = l == 1 ? g.n - 2 : g.h;
    if ((t - 2 * L - 2) % 2 == 0) {
      kind = MK_NONE;
      row = (int)(local / in);
      col = (int)(local % in);
    } else {
      kind = -1;
      row = (int)local;
      col = 0;
    }
    return;
  }
  if (g.phase_mode && t >= 4 * L + 2) t -= 2 * L;   // the phase head, as a head below
  if (t < 2 * L) {
    const int l = t / 2;
    in = l == 0 ? g.n : g.h;
    if (t % 2 == 0) {
      kind = l == 0 ? MK_L1 : MK_HID;
      row = (int)(local / in);
      col = (int)(local % in);
    } else {
      kind = -1;
      row = (int)local;
      col = 0;
    }
  } else {
    const int k = t - 2 * L;   // 0 W_o, 1 b_o, 2 W_p, 3 b_p
    in = g.h;
    if (k == 0 || k == 2) {
      kind = k == 0 ? MK_HEAD_O : (g.phase_mode ? MK_NONE : MK_HEAD_P);
      row = (int)(local / g.h);
      col = (int)(local % g.h);
    } else {
      kind = -1;
      row = (int)local;
      col = 0;
    }
  }
}

__device__ __forceinline__ unsigned short rne_bf16(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

// With BF16 weights (P_BF16W) the network's weights are the parameters
// rounded to BF16; the backward differentiates that network.
template <typename T>
__global__ void pack_masked_kernel(Geom g, const float* __restrict__ params, T* __restrict__ wm) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= g.n_params) return;
  int tensor, kind, row, col, in;
  locate(g, p, tensor, kind, row, col, in);
  float v = params[p];
  if (kind >= 0 && g.prec == P_BF16W) v = __uint_as_float(((unsigned)rne_bf16(v)) << 16);
  wm[p] = (kind < 0 || mask_at(g, kind, row, col)) ? (T)v : (T)0;
}

void launch_pack_masked(const Geom& g, const float* params, void* wm, hipStream_t s) {
  const unsigned blocks = (unsigned)((g.n_params + 255) / 256);
  if (g.prec == P_F64)
    hipLaunchKernelGGL(pack_masked_kernel<double>, dim3(blocks), dim3(256), 0, s, g, params, (double*)wm);
  else
    hipLaunchKernelGGL(pack_masked_kernel<float>, dim3(blocks), dim3(256), 0, s, g, params, (float*)wm);
}

// ---------------------------------------------------- fused-kernel packing
// One wave packs a fragment of TB sorted rows, each lane E consecutive columns
// of its row; after the fragments, threads pack the biases.  A row is a stretch
// of weights up to `lim`; sorted units are visited class by class, original
// unit after original unit n - 1 apart, so a lane divides once for its row and
// once for its first column.  700 fragments (44 qubits, L = 3, 512 units) are
// less than a wave per SIMD: bound by the chain from index to load.  7 us; with
// each element located by itself, blocks searched one by one and the biases in
// a launch of their own 25 us.
__device__ __forceinline__ int block_of(const int* __restrict__ off, int blocks, long long local, int lane) {
  int blk = 0;   // the last block that starts at or before `local`
  for (int b0 = 1; b0 <= blocks; b0 += 64)
    blk += __popcll(__ballot(b0 + lane <= blocks && local >= off[min(b0 + lane, blocks)]));
  return blk;
}

template <int P>
__global__ __launch_bounds__(256) void pack_fused_kernel(Geom g, const float* __restrict__ params,
                                                         uint4* __restrict__ out, void* __restrict__ bias) {
  constexpr bool B16 = P == P_BF16 || P == P_BF16X3 || P == P_BF16W;
  constexpr int TB = P == P_F64 ? 16 : 32, E = B16 ? 8 : P == P_F32 ? 4 : 2, KSTEP = E * 64 / TB;
  const int n = g.n, h = g.h;
  const int frag_blocks = (int)((g.nfrag + 3) / 4);
  if ((int)blockIdx.x >= frag_blocks) {
    using S = typename std::conditional<P == P_F64, double, float>::type;
    const long long i = (long long)(blockIdx.x - frag_blocks) * 256 + threadIdx.x;
    const long long nh = (long long)g.L * h;
    if (i >= nh + (long long)g.NHB * g.TB) return;
    S v = 0;
    if (i < nh) {
      const int l = (int)(i / h), u = (int)(i % h);
      v = (S)(g.net_kind == 2 ? params[g.poff[poff_phase_layer(g, l + 1) + 1] + u]
                              : params[g.poff[2 * l + 1] + orig_of_sorted(g, u)]);
    } else {
      const int t = (int)(i - nh);
      if (g.net_kind == 2) {
        if (t < 4) v = (S)params[g.poff[poff_phase_head(g) + 1] + t];
      } else if (t < n) {
        v = (S)params[g.poff[2 * g.L + 1] + g.order[t]];
      } else if (t < n + 4 && g.net_kind == 0) {
        v = (S)params[g.poff[poff_phase_head(g) + 1] + (t - n)];
      }
    }
    ((S*)bias)[i] = v;
    return;
  }
  const int lane = threadIdx.x & 63;
  const long long f = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (f >= g.nfrag) return;
  // the fragment's block and k step, then the lane's row: its weights, the first masked column
  const int row_l = lane % TB, kofs = E * (lane / TB);
  int k0, lim = 0;
  const float* w = params;
  enum { POSITIONS, UNITS, PLAIN } cols;
  if (f < g.frag_h) {                    // layer 1: sorted units x positions
    const int blk = block_of(g.off1, g.NB, f, lane), row = TB * blk + row_l;
    k0 = KSTEP * (int)(f - g.off1[blk]) + kofs;
    if (g.net_kind == 2) {               // (separate phase network: dense, units in their own order)
      cols = PLAIN;
      lim = row < h ? n - 2 : 0;
      w += g.poff[poff_phase_layer(g, 1)] + (long long)row * (n - 2);
    } else {
      cols = POSITIONS;
      if (row < h) {
        lim = min(n, class_of_sorted(g, row) + 1);
        w += g.poff[0] + (long long)orig_of_sorted(g, row) * n;
      }
    }
  } else if (f < g.frag_head) {          // hidden layers 2..L
    const long long per = g.offh[g.NB];
    const int layer = 2 + (int)((f - g.frag_h) / per);
    const long long local = (f - g.frag_h) % per;
    const int blk = block_of(g.offh, g.NB, local, lane), row = TB * blk + row_l;
    k0 = KSTEP * (int)(local - g.offh[blk]) + kofs;
    if (g.net_kind == 2) {
      cols = PLAIN;
      lim = row < h ? h : 0;
      w += g.poff[poff_phase_layer(g, layer)] + (long long)row * h;
    } else {
      cols = UNITS;
      if (row < h) {
        lim = min(h, prefix_of_class(g, class_of_sorted(g, row) + 1));
        w += g.poff[2 * (layer - 1)] + (long long)orig_of_sorted(g, row) * h;
      }
    }
  } else {                               // head: positions 0..n-1, then 4 phase rows
    const long long local = f - g.frag_head;
    const int blk = block_of(g.offo, g.NHB, local, lane), row = TB * blk + row_l;
    k0 = KSTEP * (int)(local - g.offo[blk]) + kofs;
    cols = g.net_kind == 2 ? PLAIN : UNITS;
    if (g.net_kind == 2) {
      lim = row < 4 ? h : 0;
      w += g.poff[poff_phase_head(g)] + (long long)row * h;
    } else if (row < n) {
      lim = min(h, prefix_of_class(g, row));
      w += g.poff[2 * g.L] + (long long)g.order[row] * h;
    } else if (row < n + 4 && g.net_kind == 0) {
      lim = min(h, prefix_of_class(g, n - 2));
      w += g.poff[poff_phase_head(g)] + (long long)(row - n) * h;
    }
  }
  float v[E];
  int c = 0, o = k0;                     // UNITS: class and original unit of column k0
  if (cols == UNITS) {
    c = class_of_sorted(g, min(k0, h - 1));
    o = c + (min(k0, h - 1) - prefix_of_class(g, c)) * (n - 1);
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const bool in = k0 + j < lim;
    v[j] = in ? w[cols == POSITIONS ? (int)g.order[in ? k0 + j : 0] : o] : 0.f;
    if (cols == UNITS) {
      const bool same = o + n - 1 < h;
      c += same ? 0 : 1;
      o = same ? o + n - 1 : c;
    } else {
      o += 1;
    }
  }
  uint4 hi, lo = make_uint4(0, 0, 0, 0);
  if constexpr (B16) {
    unsigned vh[8], vl[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      vh[j] = rne_bf16(v[j]);
      vl[j] = rne_bf16(v[j] - __uint_as_float(vh[j] << 16));
    }
    hi = make_uint4(vh[0] | (vh[1] << 16), vh[2] | (vh[3] << 16), vh[4] | (vh[5] << 16), vh[6] | (vh[7] << 16));
    lo = make_uint4(vl[0] | (vl[1] << 16), vl[2] | (vl[3] << 16), vl[4] | (vl[5] << 16), vl[6] | (vl[7] << 16));
  } else if constexpr (P == P_F32) {
    hi = __builtin_bit_cast(uint4, make_float4(v[0], v[1], v[2], v[3]));
  } else {
    hi = __builtin_bit_cast(uint4, make_double2((double)v[0], (double)v[1]));
  }
  out[f * 64 + lane] = hi;
  if (g.planes == 2) out[(g.nfrag + f) * 64 + lane] = lo;
}

void launch_pack_fused(const Geom& g, const float* params, void* packed, hipStream_t s) {
  const long long nb = (long long)g.L * g.h + (long long)g.NHB * g.TB;
  const dim3 grid((unsigned)((g.nfrag + 3) / 4 + (nb + 255) / 256)), block(256);
  void* bias = (char*)packed + g.bias_byte;
  auto kern = g.prec == P_F64 ? pack_fused_kernel<P_F64> : g.prec == P_F32 ? pack_fused_kernel<P_F32>
                                                                           : pack_fused_kernel<P_BF16>;
  hipLaunchKernelGGL(kern, grid, block, 0, s, g, params, (uint4*)packed, bias);
}

// ------------------------------------------------------------ small GEMM
// C(i,j) = sum_k A(i,k) B(k,j) in 64x64 tiles, 256 threads.  What is contiguous
// in memory follows from the use: activations and seeds are rows of samples.
//   E_FWD      relu(A B + bias)    A by k, B by k   (activations x weights^T)
//   E_FWD_LIN  A B + bias          A by k, B by k
//   E_STORE    A B                 A by k, B by j   (seeds x weights)
//   E_ADD      C + A B             A by k, B by j
//   E_GRAD     grad += A B         A by i, B by j   (seeds^T x activations, k = samples)
// E_STORE and E_ADD take the derivative of the ReLU in front of C (act) along.
//
// E_GRAD sums over the samples.  They are cut into blocks of KBLK: a block's
// products are summed by one chain in the path's type and the blocks in order
// in FP64.  With room for the blocks' sums (part) every block is a workgroup of
// its own and a second kernel adds them; without it one workgroup takes them
// in turn.  Both give the same bits.  The sums are bound by how many workgroups
// a [h][h] result has: one chain over 4,096 samples ran 64 workgroups at 512
// units for 480 us (16 at 256 units, 485 us); blocks take 20 us (14 us) and
// their reduction 6 us, and the FP32 chains are 16 times shorter.  The same
// workgroups sum A over the samples for the biases (a kernel of 45 us before).
enum Epi { E_FWD = 0, E_FWD_LIN = 1, E_STORE = 2, E_ADD = 3, E_GRAD = 4 };

struct GemmArgs {
  int Mr, Nc, K;
  const void* A; long long sa;   // stride of A's and B's rows in memory
  const void* B; long long sb;
  void* C; long long ldc;
  const void* bias;        // E_FWD / E_FWD_LIN
  const void* act;         // E_STORE / E_ADD: C is 0 where act (ldc) is not positive; nullptr: everywhere kept
  double* grad; long long grad_off, bias_off; int mask_kind;   // E_GRAD: rows of Nc, biases
  void* part;              // E_GRAD: sums of the blocks [nz][Mr][Nc], then of A over the block [nz][Mr] FP64
  int z0, nz;              // E_GRAD: blocks z0 .. z0 + nz - 1
};

template <typename T> constexpr int kblk() { return sizeof(T) == 4 ? 256 : 64; }

// Sums of A over the samples of block z behind the blocks' sums.
template <typename T>
__device__ __forceinline__ double* part_bias(const GemmArgs& a) {
  return (double*)((char*)a.part + (((size_t)a.nz * a.Mr * a.Nc * sizeof(T) + 15) & ~(size_t)15));
}

// The tile of C at (i0, j0): lane's elements are given by (row, col) pairs.
template <typename T, int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, int i, int j, T v) {
  if (i >= a.Mr || j >= a.Nc) return;
  T* c = (T*)a.C + i * a.ldc + j;
  if constexpr (EPI == E_FWD || EPI == E_FWD_LIN) {
    v += ((const T*)a.bias)[j];
    if (EPI == E_FWD) v = v > (T)0 ? v : (T)0;
    *c = v;
  } else {
    if constexpr (EPI == E_ADD) v += *c;
    if (a.act && !(((const T*)a.act)[i * a.ldc + j] > (T)0)) v = (T)0;
    *c = v;
  }
}

// One element of E_GRAD: its block's sum, or (no room for the blocks) the
// total of all of them.
template <typename T>
__device__ __forceinline__ void grad_store(const GemmArgs& a, const Geom& g, int z, int i, int j, T v, double total) {
  if (i >= a.Mr || j >= a.Nc) return;
  if (a.part) ((T*)a.part)[((size_t)z * a.Mr + i) * a.Nc + j] = v;
  else if (mask_at(g, a.mask_kind, i, j)) a.grad[a.grad_off + (long long)i * a.Nc + j] = total;
}
__device__ __forceinline__ double grad_before(const GemmArgs& a, const Geom& g, int i, int j) {
  return !a.part && i < a.Mr && j < a.Nc && mask_at(g, a.mask_kind, i, j)
             ? a.grad[a.grad_off + (long long)i * a.Nc + j] : 0.0;
}

// Sum of A's rows i0 + t over the 16 or 32 staged samples (threads t < 64).
template <typename T, int BK, int LD>
__device__ __forceinline__ double stage_sum(const T (&As)[BK][LD], int t) {
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < BK; ++k) s += (double)As[k][t];
  return s;
}

// Blocks summed in order onto the gradient: weights, then biases.
template <typename T>
__global__ __launch_bounds__(256) void grad_reduce_kernel(GemmArgs a, Geom g) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long n = (long long)a.Mr * a.Nc;
  if (e < n) {
    const int i = (int)(e / a.Nc), j = (int)(e % a.Nc);
    if (!mask_at(g, a.mask_kind, i, j)) return;
    double t = a.grad[a.grad_off + e];
    for (int z = 0; z < a.nz; ++z) t += (double)((const T*)a.part)[z * n + e];
    a.grad[a.grad_off + e] = t;
  } else if (e < n + a.Mr) {
    const int i = (int)(e - n);
    const double* pb = part_bias<T>(a);
    double t = a.grad[a.bias_off + i];
    for (int z = 0; z < a.nz; ++z) t += pb[(long long)z * a.Mr + i];
    a.grad[a.bias_off + i] = t;
  }
}

// FP64: 16 samples or k at a time through LDS, 4x4 elements per thread.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f64_kernel(GemmArgs a, Geom g) {
  typedef double T;
  __shared__ T As[16][65];
  __shared__ T Bs[16][65];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  const T* A = (const T*)a.A;
  const T* B = (const T*)a.B;
  const int nblk = EPI == E_GRAD ? (a.part ? 1 : a.nz) : 1;
  double total[4][4], bsum = 0.0;
  if constexpr (EPI == E_GRAD) {
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) total[p][q] = grad_before(a, g, i0 + ty + 16 * p, j0 + tx + 16 * q);
  }
  T acc[4][4] = {};
  const int bz = EPI == E_GRAD && a.part ? (int)blockIdx.z : 0;
  for (int z = bz; z < bz + nblk; ++z) {
    const int kb = EPI == E_GRAD ? (a.z0 + z) * kblk<T>() : 0;
    const int ke = EPI == E_GRAD ? min(a.K, kb + kblk<T>()) : a.K;
    double bz_sum = 0.0;
    for (int k0 = kb; k0 < ke; k0 += 16) {
      for (int e = threadIdx.x; e < 1024; e += 256) {
        const int r = EPI == E_GRAD ? e & 63 : e >> 4, kk = EPI == E_GRAD ? e >> 6 : e & 15;   // A: 64 rows x 16 k
        const int gi = i0 + r, gk = k0 + kk;
        As[kk][r] = (gi < a.Mr && gk < ke) ? (EPI == E_GRAD ? A[gk * a.sa + gi] : A[gi * a.sa + gk]) : 0.0;
        constexpr bool BK_ = EPI == E_FWD || EPI == E_FWD_LIN;
        const int kb2 = BK_ ? e & 15 : e >> 6, c = BK_ ? e >> 4 : e & 63;                      // B: 16 k x 64 cols
        const int gkb = k0 + kb2, gj = j0 + c;
        Bs[kb2][c] = (gkb < ke && gj < a.Nc) ? (BK_ ? B[gj * a.sb + gkb] : B[gkb * a.sb + gj]) : 0.0;
      }
      __syncthreads();
      if (EPI == E_GRAD && blockIdx.x == 0 && threadIdx.x < 64) bz_sum += stage_sum(As, threadIdx.x);
#pragma unroll
      for (int kk = 0; kk < 16; ++kk) {
        T av[4], bv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) { av[q] = As[kk][ty + 16 * q]; bv[q] = Bs[kk][tx + 16 * q]; }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[p][q] += av[p] * bv[q];
      }
      __syncthreads();
    }
    if constexpr (EPI == E_GRAD) {
      if (a.part) {
        if (blockIdx.x == 0 && threadIdx.x < 64 && i0 + (int)threadIdx.x < a.Mr)
          part_bias<T>(a)[(long long)z * a.Mr + i0 + threadIdx.x] = bz_sum;
      } else {
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int q = 0; q < 4; ++q) { total[p][q] += acc[p][q]; acc[p][q] = 0.0; }
        if (z == 0 && i0 + (int)threadIdx.x < a.Mr && threadIdx.x < 64) bsum = a.grad[a.bias_off + i0 + threadIdx.x];
        bsum += bz_sum;
      }
    }
  }
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + ty + 16 * p, j = j0 + tx + 16 * q;
      if constexpr (EPI == E_GRAD) grad_store<T>(a, g, bz, i, j, acc[p][q], total[p][q]);
      else gemm_epilogue<T, EPI>(a, i, j, acc[p][q]);
    }
  if (EPI == E_GRAD && !a.part && blockIdx.x == 0 && threadIdx.x < 64 && i0 + (int)threadIdx.x < a.Mr)
    a.grad[a.bias_off + i0 + threadIdx.x] = bsum;
}

// FP32 on the matrix cores: 32 k at a time through LDS, the next 32 already
// requested; each of the four waves owns a 32x32 quarter of the tile and
// accumulates it with v_mfma_f32_32x32x2f32 (lane l supplies A row l % 32 and B
// column l % 32 at k = l / 32; accumulator r of lane l holds row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of the quarter).
typedef __attribute__((ext_vector_type(16))) float gemm_f32x16;

// 32 k x 64 lines of a tile, 8 values per thread.  KC: lines are contiguous
// along k (a thread takes 8 k of one line), else along the lines (8 lines of
// one k).  Tensors of the flat layout start at any multiple of 4 bytes, which
// is the alignment that four-float loads need here.
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
template <bool KC>
struct TileLoad {
  static constexpr int LD = KC ? 66 : 68;   // LDS row: no bank conflicts for the stores of either form
  float v[8];
  __device__ __forceinline__ void load(const float* p, long long ld, int line0, int lines, int k0, int ke) {
    const int t = threadIdx.x;
    const int line = line0 + (KC ? t >> 2 : (t & 7) * 8), k = k0 + (KC ? (t & 3) * 8 : t >> 3);
    const float* q = p + (KC ? (long long)line * ld + k : (long long)k * ld + line);
    const int n = KC ? (line < lines ? ke - k : 0) : (k < ke ? lines - line : 0);   // values in range, from the first
    if (n >= 8) {
      const float4u x = *(const float4u*)q, y = *(const float4u*)(q + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[e] = x[e]; v[4 + e] = y[e]; }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = e < n ? q[e] : 0.f;
    }
  }
  __device__ __forceinline__ void store(float (&s)[32][LD]) const {
    const int t = threadIdx.x;
    if constexpr (KC) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s[(t & 3) * 8 + e][t >> 2] = v[e];
    } else {
      *(float4*)&s[t >> 3][(t & 7) * 8] = make_float4(v[0], v[1], v[2], v[3]);
      *(float4*)&s[t >> 3][(t & 7) * 8 + 4] = make_float4(v[4], v[5], v[6], v[7]);
    }
  }
};

template <int EPI>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(GemmArgs a, Geom g) {
  constexpr bool AK = EPI != E_GRAD, BKC = EPI == E_FWD || EPI == E_FWD_LIN;
  __shared__ __align__(16) float As[32][TileLoad<AK>::LD];
  __shared__ __align__(16) float Bs[32][TileLoad<BKC>::LD];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wy = wave >> 1, wx = wave & 1;
  const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  const float* A = (const float*)a.A;
  const float* B = (const float*)a.B;
  gemm_f32x16 acc = {};
  const int li = lane & 31, lk = lane >> 5;
  const int j = j0 + wx * 32 + li;
  auto row = [&](int r) { return i0 + wy * 32 + 8 * (r >> 2) + 4 * lk + (r & 3); };
  const int nblk = EPI == E_GRAD && !a.part ? a.nz : 1;
  const int bz = EPI == E_GRAD && a.part ? (int)blockIdx.z : 0;
  double total[EPI == E_GRAD ? 16 : 1], bsum = 0.0;
  if constexpr (EPI == E_GRAD) {
#pragma unroll
    for (int r = 0; r < 16; ++r) total[r] = grad_before(a, g, row(r), j);
  }
  const bool sums = EPI == E_GRAD && blockIdx.x == 0 && threadIdx.x < 64;   // this thread sums row i0 + t of A
  const int bi = i0 + (int)threadIdx.x;
  for (int z = bz; z < bz + nblk; ++z) {
    const int kb = EPI == E_GRAD ? (a.z0 + z) * kblk<float>() : 0;
    const int ke = EPI == E_GRAD ? min(a.K, kb + kblk<float>()) : a.K;
    double block_sum = 0.0;
    TileLoad<AK> la;
    TileLoad<BKC> lb;
    la.load(A, a.sa, i0, a.Mr, kb, ke);
    lb.load(B, a.sb, j0, a.Nc, kb, ke);
    for (int k0 = kb; k0 < ke; k0 += 32) {
      la.store(As);
      lb.store(Bs);
      __syncthreads();
      if (k0 + 32 < ke) {
        la.load(A, a.sa, i0, a.Mr, k0 + 32, ke);
        lb.load(B, a.sb, j0, a.Nc, k0 + 32, ke);
      }
      if (sums) block_sum += stage_sum(As, threadIdx.x);
#pragma unroll
      for (int kk = 0; kk < 32; kk += 2)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(As[kk + lk][wy * 32 + li], Bs[kk + lk][wx * 32 + li], acc, 0, 0, 0);
      __syncthreads();
    }
    if constexpr (EPI == E_GRAD) {
      if (a.part) {
        if (sums && bi < a.Mr) part_bias<float>(a)[(long long)z * a.Mr + bi] = block_sum;
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r] += (double)acc[r];
        acc = gemm_f32x16{};
        if (sums && z == 0 && bi < a.Mr) bsum = a.grad[a.bias_off + bi];
        bsum += block_sum;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    if constexpr (EPI == E_GRAD) grad_store<float>(a, g, bz, row(r), j, acc[r], total[r]);
    else gemm_epilogue<float, EPI>(a, row(r), j, acc[r]);
  }
  if (EPI == E_GRAD && !a.part && sums && bi < a.Mr) a.grad[a.bias_off + bi] = bsum;
}

template <typename T, int EPI>
static void gemm(const GemmArgs& a, const Geom& g, hipStream_t s, unsigned blocks = 1) {
  if (a.Mr <= 0 || a.Nc <= 0) return;
  dim3 grid((unsigned)((a.Nc + 63) / 64), (unsigned)((a.Mr + 63) / 64), blocks);
  if constexpr (sizeof(T) == 4) hipLaunchKernelGGL((gemm_mfma_kernel<EPI>), grid, dim3(256), 0, s, a, g);
  else hipLaunchKernelGGL((gemm_f64_kernel<EPI>), grid, dim3(256), 0, s, a, g);
}

// E_GRAD over all blocks of a.K samples: as many blocks at once as `room` bytes
// at `part` hold the sums of.  A single block needs none.
template <typename T>
static void gemm_grad(GemmArgs a, const Geom& g, void* part, size_t room, hipStream_t s) {
  if (a.Mr <= 0 || a.Nc <= 0) return;
  const int nz = (a.K + kblk<T>() - 1) / kblk<T>();
  const size_t per = (size_t)a.Mr * a.Nc * sizeof(T) + (size_t)a.Mr * 8;
  const int fit = room > 16 ? (int)std::min<size_t>(nz, (room - 16) / per) : 0;
  if (nz <= 1 || fit < 2) {
    a.part = nullptr;
    a.z0 = 0;
    a.nz = nz;
    gemm<T, E_GRAD>(a, g, s);
    return;
  }
  a.part = part;
  for (int z = 0; z < nz; z += fit) {
    a.z0 = z;
    a.nz = std::min(fit, nz - z);
    gemm<T, E_GRAD>(a, g, s, (unsigned)a.nz);
    const long long n = (long long)a.Mr * a.Nc + a.Mr;
    hipLaunchKernelGGL(grad_reduce_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a, g);
  }
}

// Bit of qubit j of sample i (g.words 64-bit words per sample).
__device__ __forceinline__ int qubit_bit(const Geom& g, const uint64_t* __restrict__ x, long long i, int j) {
  return (int)((x[i * g.words + (j >> 6)] >> (j & 63)) & 1ull);
}

template <typename T>
__global__ void bits_kernel(Geom g, const uint64_t* __restrict__ x, long long S, T* __restrict__ s) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= S * g.n) return;
  const long long i = e / g.n;
  const int j = (int)(e % g.n);
  s[e] = qubit_bit(g, x, i, j) ? (T)1 : (T)-1;
}

// Output seeds for sample i with g_la = 2 (w/W)(Re l - E), g_phi = 2 (w/W) Im l:
// d o_j = g_la * 1/2 * free_j * (x_j - sigmoid(o_j)); d p_c = g_phi [c == sel].
template <typename T>
__global__ void seed_kernel(Geom g, const uint64_t* __restrict__ x, long long S,
                            const double* __restrict__ eloc, const double* __restrict__ w,
                            const double* __restrict__ energy, const T* __restrict__ hout,
                            T* __restrict__ dh) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= S) return;
  const int n = g.n, ld = n + 4;
  const double W = energy[2], E = energy[0];
  const double wi = w ? w[i] : 1.0;
  const double gla = 2.0 * (wi / W) * (eloc[2 * i] - E);
  const double gph = 2.0 * (wi / W) * eloc[2 * i + 1];
  const bool constrained = g.n_up >= 0 && g.n_dn >= 0;
  int placed[2] = {0, 0};
  int remaining[2] = {(int)__popcll(g.spin_pos[0]) + (int)__popcll(g.spin_pos_hi[0]),
                      (int)__popcll(g.spin_pos[1]) + (int)__popcll(g.spin_pos_hi[1])};
  for (int t = 0; t < n; ++t) {
    const int j = g.order[t];
    const int sp = j & 1;
    remaining[sp] -= 1;
    const int bit = qubit_bit(g, x, i, j);
    bool fr = true;
    if (constrained) {
      const int ns = sp ? g.n_dn : g.n_up;
      fr = !(placed[sp] >= ns || placed[sp] + remaining[sp] < ns);
    }
    placed[sp] += bit;
    const double o = (double)hout[i * ld + j];
    const double sig = 1.0 / (1.0 + exp(-o));
    dh[i * ld + j] = fr ? (T)(gla * 0.5 * ((double)bit - sig)) : (T)0;
  }
  const int sel = 2 * qubit_bit(g, x, i, g.order[n - 2]) + qubit_bit(g, x, i, g.order[n - 1]);
  for (int c = 0; c < 4; ++c) dh[i * ld + n + c] = c == sel ? (T)gph : (T)0;
}

// Input of a separate phase network: the first n-2 entries in sampling order.
template <typename T>
__global__ void phase_input_kernel(Geom g, const T* __restrict__ s, long long S, T* __restrict__ v) {
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int np = g.n - 2;
  if (e >= S * np) return;
  const long long i = e / np;
  const int t = (int)(e % np);
  v[e] = s[i * g.n + g.order[t]];
}

// Forward of L ReLU layers over S rows: acts[l] = relu(in_l W_l^T + b_l), the
// weight and bias of layer l at poff[wi(l)], poff[wi(l) + 1].
template <typename T, class WIdx>
static void mlp_forward(const Geom& g, const T* wm, const T* in0, int k0, long long S, T* acts, WIdx wi,
                        hipStream_t s) {
  const int h = g.h;
  for (int l = 1; l <= g.L; ++l) {
    const int K = l == 1 ? k0 : h;
    GemmArgs a{};
    a.Mr = (int)S; a.Nc = h; a.K = K;
    a.A = l == 1 ? (const void*)in0 : (const void*)(acts + (long long)(l - 2) * S * h);
    a.sa = K;
    a.B = wm + g.poff[wi(l)]; a.sb = K;
    a.C = acts + (long long)(l - 1) * S * h; a.ldc = h;
    a.bias = wm + g.poff[wi(l) + 1];
    gemm<T, E_FWD>(a, g, s);
  }
}

// Reverse pass through those layers from d(acts[L]), already past the last
// ReLU, in da: gradients of the weights (masked by mask_of(l)) and biases; da
// and dz are S x h scratch.
template <typename T, class WIdx, class MIdx>
static void mlp_backward(const Geom& g, const T* wm, const T* in0, int k0, long long S, const T* acts, T* da,
                         T* dz, double* grad, void* part, size_t room, WIdx wi, MIdx mask_of, hipStream_t s) {
  const int h = g.h;
  for (int l = g.L; l >= 1; --l) {
    const int K = l == 1 ? k0 : h;
    const T* prev = l == 1 ? in0 : acts + (long long)(l - 2) * S * h;
    GemmArgs a{};
    a.Mr = h; a.Nc = K; a.K = (int)S;
    a.A = da; a.sa = h;
    a.B = prev; a.sb = K;
    a.grad = grad; a.grad_off = g.poff[wi(l)]; a.bias_off = g.poff[wi(l) + 1];
    a.mask_kind = mask_of(l);
    gemm_grad<T>(a, g, part, room, s);
    if (l > 1) {
      GemmArgs b{};
      b.Mr = (int)S; b.Nc = K; b.K = h;
      b.A = da; b.sa = h;
      b.B = wm + g.poff[wi(l)]; b.sb = K;
      b.C = dz; b.ldc = K;
      b.act = prev;
      gemm<T, E_STORE>(b, g, s);
      T* t = da; da = dz; dz = t;
    }
  }
}

template <typename T>
static void backward_t(const Geom& g, const T* wm, const uint64_t* x, long long S, const double* eloc,
                       const double* w, const double* energy, T* scratch, double* grad, void* part, size_t room,
                       hipStream_t s) {
  const int n = g.n, h = g.h, L = g.L, ld = n + 4;
  const bool two = g.phase_mode == 1;
  T* sb = scratch;
  T* acts = sb + S * n;
  T* hout = acts + (long long)L * S * h;
  T* dh = hout + S * ld;
  T* da = dh + S * ld;
  T* dz = da + S * h;
  T* pin = dz + S * h;                     // separate phase network: input and activations
  T* pacts = pin + S * (n - 2);
  const unsigned eb = (unsigned)((S * n + 255) / 256);
  hipLaunchKernelGGL(bits_kernel<T>, dim3(eb), dim3(256), 0, s, g, x, S, sb);
  // forward recompute
  auto trunk_w = [&](int l) { return 2 * (l - 1); };
  auto phase_w = [&](int l) { return poff_phase_layer(g, l); };
  mlp_forward<T>(g, wm, sb, n, S, acts, trunk_w, s);
  const T* aL = acts + (long long)(L - 1) * S * h;
  const T* phin = aL;                      // what the phase head reads
  if (two) {
    const long long ne = S * (n - 2);
    hipLaunchKernelGGL(phase_input_kernel<T>, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, s, g,
                       (const T*)sb, S, pin);
    mlp_forward<T>(g, wm, pin, n - 2, S, pacts, phase_w, s);
    phin = pacts + (long long)(L - 1) * S * h;
  }
  const int hw[2] = {2 * L, poff_phase_head(g)};
  for (int head = 0; head < 2; ++head) {
    GemmArgs a{};
    a.Mr = (int)S; a.Nc = head == 0 ? n : 4; a.K = h;
    a.A = head == 0 ? aL : phin; a.sa = h;
    a.B = wm + g.poff[hw[head]]; a.sb = h;
    a.C = hout + (head == 0 ? 0 : n); a.ldc = ld;
    a.bias = wm + g.poff[hw[head] + 1];
    gemm<T, E_FWD_LIN>(a, g, s);
  }
  hipLaunchKernelGGL(seed_kernel<T>, dim3((unsigned)((S + 255) / 256)), dim3(256), 0, s, g, x, S, eloc, w,
                     energy, hout, dh);
  // head gradients
  for (int head = 0; head < 2; ++head) {
    GemmArgs a{};
    a.Mr = head == 0 ? n : 4; a.Nc = h; a.K = (int)S;
    a.A = dh + (head == 0 ? 0 : n); a.sa = ld;
    a.B = head == 0 ? aL : phin; a.sb = h;
    a.grad = grad; a.grad_off = g.poff[hw[head]]; a.bias_off = g.poff[hw[head] + 1];
    a.mask_kind = head == 0 ? MK_HEAD_O : (two ? MK_NONE : MK_HEAD_P);
    gemm_grad<T>(a, g, part, room, s);
  }
  // d a_L = d o (M_o W_o) [+ d p (M_p W_p) with the shared trunk], through the last ReLU
  {
    GemmArgs a{};
    a.Mr = (int)S; a.Nc = h; a.K = n;
    a.A = dh; a.sa = ld;
    a.B = wm + g.poff[2 * L]; a.sb = h;
    a.C = da; a.ldc = h;
    a.act = two ? aL : nullptr;
    gemm<T, E_STORE>(a, g, s);
    if (!two) {
      a.K = 4;
      a.A = dh + n;
      a.B = wm + g.poff[hw[1]];
      a.act = aL;
      gemm<T, E_ADD>(a, g, s);
    }
  }
  mlp_backward<T>(g, wm, sb, n, S, acts, da, dz, grad, part, room, trunk_w,
                  [&](int l) { return l == 1 ? (int)MK_L1 : (int)MK_HID; }, s);
  if (two) {
    // d c_L = d p W_p, then through the phase network's dense layers
    GemmArgs a{};
    a.Mr = (int)S; a.Nc = h; a.K = 4;
    a.A = dh + n; a.sa = ld;
    a.B = wm + g.poff[hw[1]]; a.sb = h;
    a.C = da; a.ldc = h;
    a.act = phin;
    gemm<T, E_STORE>(a, g, s);
    mlp_backward<T>(g, wm, pin, n - 2, S, pacts, da, dz, grad, part, room, phase_w, [&](int) { return (int)MK_NONE; },
                    s);
  }
}

long long backward_scratch_elems(const Geom& g, long long S) {
  long long e = S * (long long)(g.n + (long long)g.L * g.h + 2 * (g.n + 4) + 2 * g.h);
  if (g.phase_mode == 1) e += S * (long long)((g.n - 2) + (long long)g.L * g.h);
  return e;
}

void launch_backward(const Geom& g, const void* wm, const uint64_t* x, long long S,
                     const double* eloc, const double* w, const double* energy, void* scratch,
                     double* grad, void* part, size_t room, hipStream_t s) {
  if (S <= 0) return;
  if (g.prec == P_F64)
    backward_t<double>(g, (const double*)wm, x, S, eloc, w, energy, (double*)scratch, grad, part, room, s);
  else
    backward_t<float>(g, (const float*)wm, x, S, eloc, w, energy, (float*)scratch, grad, part, room, s);
}

}  // namespace nqs
