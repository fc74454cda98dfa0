// Prefix-shared forward of the connected configurations.
//
// The masks of Sec. 4 make a hidden unit of degree d a function of the first
// d sampling positions only, and the enumeration lists a sample's connected
// configurations flip by ascending flip, which in the default (reverse)
// sampling order is a depth-first walk of their binary prefix tree: at 60
// qubits consecutive configurations share 11 rows per distinct prefix of 30
// positions and 2.4 per prefix of 45.  So the network is not evaluated row by
// row but down that tree.  Units sorted by degree are cut at a few blocks
// (the levels); a node is a distinct prefix of the positions its level's
// units depend on.  For the nodes of a level the kernel
//   * evaluates that level's own units in every layer (their inputs are the
//     level's own units and, through the parent's state, all earlier ones);
//   * multiplies them into the pre-activations of every later unit and head
//     row, once per node instead of once per row: the node's state;
//   * adds the log-sigmoids of the positions that are complete.
// The last level's nodes are the rows.  Per weight pair the work is one
// product per distinct prefix of the earlier unit: at 60 qubits with cuts at
// 1/4, 1/2 and 3/4 of 1024 units a sixth of the row-by-row forward's.
//
// Each pre-activation is the same chain of MFMAs in the same k order as in the
// row-by-row kernel (a state is a chain interrupted at a block boundary and
// carried in the accumulator's own type; the head's k slices are carried as
// the sum of the finished slices and the slice in progress), and both kernels
// add the log-sigmoids in one order, so log|psi| and phi are that kernel's,
// bit for bit.
//
// A workgroup of eight waves walks its own segment of rows depth first, a tile
// of M nodes at a time, and keeps two tiles of states per level, so states need
// room per workgroup and not for every node of the call.  Two workgroups share
// a CU and fill each other's barriers (one alone takes 1.26 times as long).  At
// 60 qubits and 1024 units the matrix cores are busy 33% of the time, beside
// state traffic of 3.5 TB/s past L2; at 64 qubits and 512 units 20%, where the
// vector instructions of the conversions and the log-sigmoids take half of the
// issue cycles and the activations' reads most of LDS's rate during the products.
// Measured on 2,000 samples at 60 qubits, L = 4, 1024 units: 191 ms against
// 610 ms row by row; 8,192 samples at 40 qubits, L = 3, 512 units: 32 ms against
// 88 ms; 400 samples (38 million rows) at 64 qubits: 27.6 ms against 63 ms.
#include <algorithm>
#include <atomic>

#include "nqs_internal.h"

namespace nqs {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int kWaves = 8, kThreads = 64 * kWaves;

// Per arithmetic kind: MFMA block TB, k per fragment, activation and weight
// planes (hi, lo), the row blocks RB of a wave's tile and the tiles a wave may
// hold between two barriers.  A tile of two row blocks takes each weight
// fragment from L2 once; FP32 and FP64 MFMAs run 8 and more times as long per
// fragment, so there single tiles, which spread over the waves more evenly.
template <int P> struct Kind;
template <> struct Kind<P_BF16>   { static constexpr int TB = 32, KSTEP = 16, PL = 1, PLW = 1, RB = 2, SLOTS = 2; using Acc = f32x16; using S = float; };
template <> struct Kind<P_BF16X3> { static constexpr int TB = 32, KSTEP = 16, PL = 2, PLW = 2, RB = 2, SLOTS = 2; using Acc = f32x16; using S = float; };
template <> struct Kind<P_BF16W>  { static constexpr int TB = 32, KSTEP = 16, PL = 2, PLW = 1, RB = 2, SLOTS = 2; using Acc = f32x16; using S = float; };
template <> struct Kind<P_F32>    { static constexpr int TB = 32, KSTEP = 8, PL = 1, PLW = 1, RB = 1, SLOTS = 4; using Acc = f32x16; using S = float; };
template <> struct Kind<P_F64>    { static constexpr int TB = 16, KSTEP = 8, PL = 1, PLW = 1, RB = 1, SLOTS = 5; using Acc = f64x4; using S = double; };

// A tile of MB row blocks: two, whose row blocks share a wave's weight
// fragments, or one, where whole tiles would leave CUs without one (the
// sampler's smaller buffers).
template <int P, int MB> struct Shape {
  static constexpr int M = MB * Kind<P>::TB;
  static constexpr int RB = MB == 2 ? Kind<P>::RB : 1;
  static constexpr int SLOTS = MB == 2 ? Kind<P>::SLOTS : P == P_F64 ? 3 : 2;
};

// One product of a weight and an activation fragment; AX: the activations are
// exact in BF16 (the +-1 inputs), their low plane is zero.
template <int P, bool AX>
__device__ __forceinline__ void mma(typename Kind<P>::Acc& acc, const uint4* w, const uint4* a) {
  if constexpr (P == P_F64) {
    const double2 wd = __builtin_bit_cast(double2, w[0]), ad = __builtin_bit_cast(double2, a[0]);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wd.x, ad.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(wd.y, ad.y, acc, 0, 0, 0);
  } else if constexpr (P == P_F32) {
    const float4 wf = __builtin_bit_cast(float4, w[0]), af = __builtin_bit_cast(float4, a[0]);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.x, af.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.y, af.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.z, af.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wf.w, af.w, acc, 0, 0, 0);
  } else {
    const bf16x8 wh = __builtin_bit_cast(bf16x8, w[0]), ah = __builtin_bit_cast(bf16x8, a[0]);
    if constexpr (P == P_BF16X3)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[1]), ah, acc, 0, 0, 0);
    if constexpr (P != P_BF16 && !AX)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, __builtin_bit_cast(bf16x8, a[1]), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh, ah, acc, 0, 0, 0);
  }
}

// Packed weights: raw buffer loads of 1 KB fragments (range-checked against
// the packed buffer), one lane offset, a scalar offset per fragment.
struct Weights {
  __amdgpu_buffer_rsrc_t rsrc;
  int plane;   // bytes to the low plane
  int voff;    // lane * 16
};
__device__ __forceinline__ Weights weights(const Geom& g, const void* packed) {
  return Weights{__builtin_amdgcn_make_buffer_rsrc((void*)packed, (short)0, (int)g.bias_byte, 0x00020000),
                 (int)(g.nfrag * 1024), 0};
}
template <int P>
__device__ __forceinline__ void wload(const Weights& b, int soff, uint4 (&w)[Kind<P>::PLW]) {
  w[0] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(b.rsrc, b.voff, soff, 0));
  if constexpr (Kind<P>::PLW == 2)
    w[1] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(b.rsrc, b.voff, soff + b.plane, 0));
}

// The thread index, opaque to the optimizer: what each phase of a tile derives
// from it is formed anew there.  Otherwise every address of every phase is
// hoisted out of the walk and, at 128 registers a wave, spilled.
__device__ __forceinline__ int thread_index() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// A barrier for data in LDS: unlike __syncthreads it leaves global loads and
// stores in flight, so fragments and states can be requested ahead of it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// k steps [k0, kend) (an even number) of one unit block by the row blocks
// mb .. mb + RB - 1.  Weight fragments are requested two steps ahead.  The
// activation fragments of a product are read while the one before it is
// multiplied (the barriers keep that order: left alone, the compiler reads each
// right before its MFMA and every MFMA waits for LDS).
template <int P, int RB, bool AX, class ActFn>
__device__ __forceinline__ void strip(typename Kind<P>::Acc (&acc)[RB], const Weights& wb, int base, int mb,
                                      int k0, int kend, ActFn act) {
  uint4 wa[Kind<P>::PLW], wc[Kind<P>::PLW], f0[Kind<P>::PL], f1[Kind<P>::PL];
  auto step = [&](uint4 (&w)[Kind<P>::PLW], int k, uint4 (&f)[Kind<P>::PL], uint4 (&g)[Kind<P>::PL]) {
    if constexpr (RB == 2) {
      act(mb + 1, k, g);
      __builtin_amdgcn_sched_barrier(0);
      mma<P, AX>(acc[0], w, f);
      __builtin_amdgcn_sched_barrier(0);
      act(mb, min(k + 1, kend - 1), f);
      __builtin_amdgcn_sched_barrier(0);
      mma<P, AX>(acc[1], w, g);
    } else {
      act(mb, min(k + 1, kend - 1), g);
      __builtin_amdgcn_sched_barrier(0);
      mma<P, AX>(acc[0], w, f);
    }
    __builtin_amdgcn_sched_barrier(0);
    wload<P>(wb, base + min(k + 2, kend - 1) * 1024, w);
    __builtin_amdgcn_sched_barrier(0);
  };
  wload<P>(wb, base + k0 * 1024, wa);
  wload<P>(wb, base + (k0 + 1) * 1024, wc);
  act(mb, k0, f0);
  __builtin_amdgcn_sched_barrier(0);
  for (int k = k0; k < kend; k += 2) {
    step(wa, k, f0, f1);
    if constexpr (RB == 2) step(wc, k + 1, f0, f1);
    else step(wc, k + 1, f1, f0);
  }
}

// +-1 input fragment of row block mb, k step ks.  Positions beyond n read a
// clear bit; their weights are zero.
template <int P, int W>
__device__ __forceinline__ uint4 input_frag(const uint64_t* y, int mb, int ks, int lane) {
  using T = Kind<P>;
  constexpr int E = 16 / (P == P_F64 ? 8 : P == P_F32 ? 4 : 2);   // elements per lane
  const int row = mb * T::TB + lane % T::TB;
  const int k0 = ks * T::KSTEP + E * (lane / T::TB);
  // a fragment's positions never straddle two words
  const uint64_t word = W == 1 ? y[row] : (k0 < 128 ? y[row * W + (k0 >> 6)] : 0ull);
  const unsigned b = W == 1 && k0 >= 64 ? 0u : (unsigned)(word >> (k0 & 63));
  // -1 with the sign bit cleared where the position is occupied
  if constexpr (P == P_F64) return make_uint4(0, 0xBFF00000u ^ ((b & 1) << 31), 0, 0xBFF00000u ^ ((b & 2) << 30));
  else if constexpr (P == P_F32)
    return make_uint4(0xBF800000u ^ (b << 31), 0xBF800000u ^ ((b & 2) << 30), 0xBF800000u ^ ((b & 4) << 29),
                      0xBF800000u ^ ((b & 8) << 28));
  else {
    unsigned u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned t = b >> (2 * j);
      u[j] = 0xBF80BF80u ^ (((t & 1) << 15) | ((t & 2) << 30));
    }
    return make_uint4(u[0], u[1], u[2], u[3]);
  }
}

// relu(acc + bias) of local block lb, row block mb into the activations, in
// the operand order of the next layer (plane: bytes to the low plane).
template <int P, int MB>
__device__ __forceinline__ void store_act(char* act, const typename Kind<P>::Acc& acc,
                                          const typename Kind<P>::S* bias, int lb, int mb, int lane, int plane) {
  using T = Kind<P>;
  const int m = lane % T::TB, g = lane / T::TB;
  if constexpr (P == P_F64) {
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int nl = g + 4 * rr;
      double t = acc[rr] + bias[16 * lb + nl];
      t = t > 0.0 ? t : 0.0;
      const int kk = nl & 7;
      *(double*)(act + (((2 * lb + (nl >> 3)) * MB + mb) * 64 + m + 16 * (kk >> 1)) * 16 + 8 * (kk & 1)) = t;
    }
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b4 = *(const float4*)(bias + 32 * lb + 8 * q + 4 * g);
      float v0 = acc[4 * q + 0] + b4.x, v1 = acc[4 * q + 1] + b4.y;
      float v2 = acc[4 * q + 2] + b4.z, v3 = acc[4 * q + 3] + b4.w;
      v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); v2 = fmaxf(v2, 0.f); v3 = fmaxf(v3, 0.f);
      if constexpr (P == P_F32) {
        *(float4*)(act + (((4 * lb + q) * MB + mb) * 64 + m + 32 * g) * 16) = make_float4(v0, v1, v2, v3);
      } else {
        char* dst = act + (((2 * lb + (q >> 1)) * MB + mb) * 64 + m + 32 * (q & 1)) * 16 + 8 * g;
        const unsigned h01 = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){v0, v1}, bf16x2));
        const unsigned h23 = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){v2, v3}, bf16x2));
        *(uint2*)dst = make_uint2(h01, h23);
        if constexpr (T::PL == 2) {
          // low term: the exact residual v - hi, rounded to BF16
          const float r0 = v0 - __uint_as_float(h01 << 16), r1 = v1 - __uint_as_float(h01 & 0xFFFF0000u);
          const float r2 = v2 - __uint_as_float(h23 << 16), r3 = v3 - __uint_as_float(h23 & 0xFFFF0000u);
          *(uint2*)(dst + plane) =
              make_uint2(__builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){r0, r1}, bf16x2)),
                         __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){r2, r3}, bf16x2)));
        }
      }
    }
  }
}

// A block of TB pre-activations x TB nodes in a level's state: unit-major in
// groups of four (FP64: single units), nodes adjacent, so a wave's loads and
// stores of neighbouring nodes are contiguous.  nodes: places per unit, unit0:
// first unit of the block.
template <int P>
__device__ __forceinline__ void state_load(typename Kind<P>::Acc& acc, const char* st, unsigned nodes, int unit0,
                                           int node, int lane) {
  const int g = lane / Kind<P>::TB;
  if constexpr (P == P_F64) {
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) acc[rr] = *(const double*)(st + ((unit0 + g + 4 * rr) * nodes + node) * 8u);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = *(const float4*)(st + ((unit0 / 4 + 2 * q + g) * nodes + node) * 16u);
      acc[4 * q] = v.x; acc[4 * q + 1] = v.y; acc[4 * q + 2] = v.z; acc[4 * q + 3] = v.w;
    }
  }
}
template <int P>
__device__ __forceinline__ void state_store(const typename Kind<P>::Acc& acc, char* st, unsigned nodes, int unit0,
                                            int node, int lane) {
  const int g = lane / Kind<P>::TB;
  if constexpr (P == P_F64) {
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) *(double*)(st + ((unit0 + g + 4 * rr) * nodes + node) * 8u) = acc[rr];
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(float4*)(st + ((unit0 / 4 + 2 * q + g) * nodes + node) * 16u) =
          make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
  }
}

template <typename S>
__device__ __forceinline__ S softplus(S z) {
  S a = z > S(0) ? z : -z;
  S m = z > S(0) ? z : S(0);
  if constexpr (sizeof(S) == 4) return m + log1pf(expf(-a));
  else return m + log1p(exp(-a));
}

// Leading sampling positions (reverse order: position p = qubit n-1-p) in
// which rows r-1 and r agree; n where they are equal.
template <int W>
__device__ __forceinline__ int common_prefix(const uint64_t* x, int r, int n) {
  if constexpr (W == 1) {
    const uint64_t d = x[r] ^ x[r - 1];
    return d ? __clzll((long long)d) - (64 - n) : n;
  } else {
    const uint64_t hi = x[2 * r + 1] ^ x[2 * r - 1], lo = x[2 * r] ^ x[2 * r - 2];
    return hi ? __clzll((long long)hi) - (128 - n) : lo ? n - 64 + __clzll((long long)lo) : n;
  }
}

// Units of one level's state: (L-1) layers of the units past the
// cut, the head's finished slices and its slice in progress (per node follow the sums of
// its log-sigmoids).
template <int P>
__host__ __device__ inline long long state_units(const Geom& g, int cb) {
  return ((long long)(g.L - 1) * (g.NB - cb) + 2LL * g.NHB) * Kind<P>::TB;
}

// LDS of a tile of M nodes.
template <int P, int W, int MB>
struct TileLds {
  using S = typename Kind<P>::S;
  static constexpr int M = Shape<P, MB>::M;
  char* act;           // activations of the level's own units, by k fragment and row block
  int plane;           // bytes to their low plane
  S* stage;            // [M][stage_ld] head outputs
  int stage_ld;
  S* blds;             // bias of the layer being finished
  S* hbl;              // bias of the head rows being finished
  uint64_t* ylds;      // the nodes' prefixes, in sampling order
  int* pidx;           // the nodes' parents: places in the parents' state
  __device__ TileLds(void* smem, int own_max, int ld) {
    act = (char*)smem;
    plane = own_max * (Kind<P>::TB / Kind<P>::KSTEP) * MB * 1024;
    stage = (S*)(act + Kind<P>::PL * plane);
    stage_ld = ld;
    blds = stage + M * ld;
    hbl = blds + own_max * Kind<P>::TB;
    ylds = (uint64_t*)(hbl + ld + 1);                          // ld is odd
    pidx = (int*)(ylds + M * W);
  }
  __device__ __forceinline__ void put_prefix(int at, const uint64_t* x, int n) const {   // reverse sampling order
    if constexpr (W == 1) {
      ylds[at] = __builtin_bitreverse64(x[0]) >> (64 - n);
    } else {
      const uint64_t r0 = __builtin_bitreverse64(x[1]), r1 = __builtin_bitreverse64(x[0]);
      const int sh = 128 - n;
      ylds[2 * at] = sh == 0 ? r0 : ((r0 >> sh) | (r1 << (64 - sh)));
      ylds[2 * at + 1] = r1 >> sh;
    }
  }
};

// What a tile evaluates: units of blocks [ca, eb) given the parents' state of
// the units before ca (pst, pn places per unit), their head products, and with
// out the chains of blocks [cb, NB) over blocks [ca, cb) and of the head into
// the state st (sn places, this tile's from place).  Head rows [r0, r1) end up
// in the stage, without bias.
struct TileJob {
  int ca, cb, eb, r0, r1;
  bool out;
  const char* pst;
  unsigned pn;
  char* st;
  unsigned sn;
  int place;
};

// early(): loads requested before the head's products, which hide their latency.
template <int P, int W, int MB, class Early>
__device__ __forceinline__ void tile_units(const Geom& g, const TileLds<P, W, MB>& t, Weights wb,
                                           const typename Kind<P>::S* biases, int ksplit, int wv, const TileJob& jb,
                                           Early early) {
  using T = Kind<P>;
  using Acc = typename T::Acc;
  using S = typename T::S;
  constexpr int TB = T::TB, KB = TB / T::KSTEP, PL = T::PL, RB = Shape<P, MB>::RB, SLOTS = Shape<P, MB>::SLOTS;
  const int tid = thread_index(), lane = tid & 63, col = lane % TB;
  wb.voff = lane * 16;
  const int L = g.L, NB = g.NB, ca = jb.ca, cb = jb.cb, eb = jb.eb;
  const int ka = ca * KB, own = eb - ca;
  const int node0 = ca > 0 ? t.pidx[col] : 0, node1 = MB == 2 && ca > 0 ? t.pidx[TB + col] : 0;
  const int pun = (NB - ca) * TB, sun = (NB - cb) * TB;        // units per layer in the parents' state and in this one
  char* act = t.act;
  auto lds_act = [&](int mb, int ks, uint4 (&f)[PL]) {
    const char* a = act + (((ks - ka) * MB + mb) * 64 + lane) * 16;
    f[0] = *(const uint4*)a;
    if constexpr (PL == 2) f[1] = *(const uint4*)(a + t.plane);
  };
  // the chain of block b, row blocks mb .., in layer l up to this level's first unit
  auto parent = [&](Acc (&acc)[RB], int l, int b, int mb) {
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      acc[i] = Acc{};
      if (ca > 0)
        state_load<P>(acc[i], jb.pst, jb.pn, (l - 2) * pun + (b - ca) * TB, (mb + i) ? node1 : node0, lane);
    }
  };
  // The own blocks' tiles are dealt out largest extent first, in a snake over
  // the waves: waves w and w + 4 share a SIMD, which then gets equal work;
  // the second workgroup of a CU starts from the other end.
  const int wd = blockIdx.x >= gridDim.x / 2 ? wv ^ 3 : wv;
  auto own_block = [&](int s, int& mb) {
    const int r = (s & 1) ? kWaves * (s + 1) - 1 - wd : kWaves * s + (wd < 4 ? wd : 11 - wd);
    mb = RB == MB ? 0 : r & 1;
    return eb - 1 - r * RB / MB;
  };

  if (tid < jb.r1 - jb.r0) t.hbl[tid] = biases[(long long)L * g.h + jb.r0 + tid];
  // the input fragments, in LDS for layer 1
  if (own > 0) {
    const int kin = g.ks1[eb - 1];
    for (int it = wv; it < MB * kin; it += kWaves)
      *(uint4*)(act + (it * 64 + lane) * 16) = input_frag<P, W>(t.ylds, it % MB, it / MB, lane);
  }
  lds_barrier();
  for (int l = 1; own > 0 && l <= L; ++l) {
    const int lbase = (int)(g.frag_h + (long long)(l - 2) * g.offh[NB]);
    const S breg = tid < own * TB ? biases[(long long)(l - 1) * g.h + ca * TB + tid] : S(0);
    Acc acc[SLOTS][RB];
    if (l == 1) {
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        int mb;
        const int b = own_block(s, mb);
#pragma unroll
        for (int i = 0; i < RB; ++i) acc[s][i] = Acc{};
        if (b >= ca)
          strip<P, RB, true>(acc[s], wb, g.off1[b] * 1024, mb, 0, g.ks1[b], [&](int rb, int ks, uint4 (&f)[PL]) {
            f[0] = *(const uint4*)(act + ((ks * MB + rb) * 64 + lane) * 16);
          });
      }
    } else {
      // later units' chains over these units, into the state
      if (jb.out) {
        for (int it = wv; it < (NB - cb) * MB / RB; it += kWaves) {
          const int b = cb + it * RB / MB, mb = RB == MB ? 0 : it & 1;
          parent(acc[0], l, b, mb);
          strip<P, RB, false>(acc[0], wb, (lbase + g.offh[b]) * 1024, mb, ka, cb * KB, lds_act);
#pragma unroll
          for (int i = 0; i < RB; ++i)
            state_store<P>(acc[0][i], jb.st, jb.sn, (l - 2) * sun + (b - cb) * TB, jb.place + (mb + i) * TB + col, lane);
        }
      }
      // the own units
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        int mb;
        const int b = own_block(s, mb);
        if (b >= ca) {
          parent(acc[s], l, b, mb);
          strip<P, RB, false>(acc[s], wb, (lbase + g.offh[b]) * 1024, mb, ka, min(g.ksh[b], eb * KB), lds_act);
        }
      }
    }
    if (tid < own * TB) t.blds[tid] = breg;
    lds_barrier();
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      int mb;
      const int b = own_block(s, mb);
      if (b >= ca) {
#pragma unroll
        for (int i = 0; i < RB; ++i) store_act<P, MB>(act, acc[s][i], t.blds, b - ca, mb + i, lane, t.plane);
      }
    }
    lds_barrier();
  }

  early();
  // head: items of one head block and one row block
  const int hun = (L - 1) * sun, phun = (L - 1) * pun;
  for (int item = wv; item < MB * g.NHB; item += kWaves) {
    const int nb = item / MB, mb = item % MB;
    if (!jb.out && (TB * (nb + 1) <= jb.r0 || TB * nb >= jb.r1)) continue;   // no row wanted
    const int kso = g.kso[nb];
    const int chunk = (((kso + ksplit - 1) / ksplit) + 7) & ~7;
    const int kstop = min(kso, (jb.out ? cb : eb) * KB);
    const int node = mb ? node1 : node0;
    Acc v{}, part{};                                           // finished slices, the slice in progress
    if (ca > 0) {
      state_load<P>(v, jb.pst, jb.pn, phun + nb * TB, node, lane);
      state_load<P>(part, jb.pst, jb.pn, phun + (g.NHB + nb) * TB, node, lane);
    }
    const int base = (int)(g.frag_head + g.offo[nb]) * 1024;
    // fragments of up to eight steps requested back to back, then consumed in order
    constexpr int D = 8 / T::PLW;
    for (int k = ka; k < kstop;) {
      const int ke = min(min(kstop, (k / chunk + 1) * chunk), k + D);
      uint4 w[D][T::PLW];
#pragma unroll
      for (int d = 0; d < D; ++d) wload<P>(wb, base + min(k + d, ke - 1) * 1024, w[d]);
      uint4 f[2][PL];
      lds_act(mb, k, f[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int d = 0; d < D; ++d)
        if (k + d < ke) {
          lds_act(mb, min(k + d + 1, ke - 1), f[(d + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          mma<P, false>(part, w[d], f[d & 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
      k = ke;
      if (ke == kso || ke % chunk == 0) {                      // a slice is finished
        v += part;
        part = Acc{};
      }
    }
    if (jb.out) {
      state_store<P>(v, jb.st, jb.sn, hun + nb * TB, jb.place + mb * TB + col, lane);
      state_store<P>(part, jb.st, jb.sn, hun + (g.NHB + nb) * TB, jb.place + mb * TB + col, lane);
    }
    v += part;
    const int m = mb * TB + col, gq = lane / TB;
    constexpr int NR = P == P_F64 ? 4 : 16;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int q = nb * TB + (P == P_F64 ? gq + 4 * r : 8 * (r >> 2) + 4 * gq + (r & 3));
      if (q >= jb.r0 && q < jb.r1) t.stage[m * t.stage_ld + q - jb.r0] = v[r];
    }
  }
  lds_barrier();
}

// Spin of the qubit at position t.
__device__ __forceinline__ int spin_at(const Geom& g, int t) {
  return (int)(((t < 64 ? g.spin_pos[1] : g.spin_pos_hi[1]) >> (t & 63)) & 1ull);
}
// Eq. modifier at position t of spin sp: ones among the earlier positions of
// that spin and its later positions force the value to 0 (f0) or 1 (f1).
template <int W>
__device__ __forceinline__ void forced(const Geom& g, uint64_t y, uint64_t yh, int t, int sp, bool& f0, bool& f1) {
  const uint64_t m0 = sp ? g.spin_pos[1] : g.spin_pos[0];
  const uint64_t low0 = t >= 64 ? ~0ull : (1ull << t) - 1;
  int before = __popcll(y & m0 & low0), rem = __popcll(m0 & ~low0);
  if constexpr (W == 2) {
    const uint64_t m1 = sp ? g.spin_pos_hi[1] : g.spin_pos_hi[0];
    const uint64_t low1 = t <= 64 ? 0ull : (1ull << (t - 64)) - 1;
    before += __popcll(yh & m1 & low1);
    rem += __popcll(m1 & ~low1);
  }
  rem -= 1;                                                    // position t itself
  const int ns = sp ? g.n_dn : g.n_up;
  f0 = before >= ns;
  f1 = before + rem < ns;
}

}  // namespace

template <int P, int W>
__global__ __launch_bounds__(kThreads, 4) void tree_forward(Geom g, TreeArgs ta) {
  using S = typename Kind<P>::S;
  constexpr int M = 2 * Kind<P>::TB;
  extern __shared__ uint4 smem[];
  const TileLds<P, W, 2> t(smem, ta.own_max, ta.stage_ld);
  int* cur = t.pidx + M, *pb = cur + 4, *tiles = cur + 8;      // the walk's cursors, per level
  int* nxt = cur + 12, *wcnt = cur + 16;                       // first row past the tile; wave counts

  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = g.n;
  const S* biases = (const S*)((const char*)ta.packed + g.bias_byte);
  const Weights wb = weights(g, ta.packed);
  char* scratch = ta.scratch + (long long)blockIdx.x * ta.scratch_wg;

  long long rows = ta.bound;
  if (ta.d_count) {
    const long long c = *ta.d_count;
    rows = c < rows ? c : rows;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && ta.prof_slot) *ta.prof_slot = rows;
  const long long seg = tree_segment(rows, gridDim.x, M);
  const long long nseg = (rows + seg - 1) / seg;

  // One tile of c nodes of level j, at nodes half .. of the level's state (rows
  // row0 .. for the last level).
  auto tile = [&](int j, int c, int half, long long row0) {
    const TreeLevel& lv = ta.lev[j];
    const bool leaf = j == ta.nlev - 1;
    const char* pst = j > 0 ? scratch + ta.lev[j - 1].st : nullptr;
    char* st = scratch + lv.st;
    // A node's state carries its log-sigmoids' sums: sum_lanes of them, one per
    // thread of the node, so that rows are added in the row-by-row forward's order
    // (400 samples at 64 qubits: 28.1 ms; with one sum per node, level by level,
    // and other bits than row by row, 28.0).  1 stands for a contradiction: no sum
    // is positive.
    constexpr int NPW = 64 / M, NSUB = kWaves * NPW;
    static_assert(NSUB == sum_lanes(P), "one sum per thread of a node");
    auto subthread = [&](int tid) {                            // the sum of the level's first position is the first wave's
      return (lv.ta + wv * NPW + (NPW > 1 ? (tid & 63) / M : 0)) & (NSUB - 1);
    };
    double sum = 0.0;
    tile_units<P, W, 2>(g, t, wb, biases, ta.ksplit, wv,
                     TileJob{lv.ca, lv.cb, lv.eb, lv.ta, leaf ? (g.net_kind == 1 ? n : n + 4) : lv.tb, !leaf, pst,
                             2 * M, st, 2 * M, half},
                     [&] {
                       const int tid = thread_index();
                       if (j > 0)
                         sum = ((const double*)(pst + state_units<P>(g, lv.ca) * (2 * M) *
                                                          (long long)sizeof(S)))[subthread(tid) * (2 * M) +
                                                                                 t.pidx[tid % M]];
                     });

    // ------------------------------------------------- log-sigmoids, phase
    // A lane takes a node and a wave every eighth position (FP64, whose tiles
    // fill half a wave: two in sixteen), so what a position asks of all nodes
    // alike (its spin, the masks of the earlier positions) is scalar work: of
    // 190 vector instructions a position and node 135 are left, 117 of them
    // log1pf.  (With a node's positions on eight lanes: 400 samples at 64
    // qubits, L = 3, 512 units, 31.4 ms, now 29.9.)
    const int tid = thread_index(), m = tid % M, sub = subthread(tid);
    const uint64_t y = t.ylds[m * W], yh = W == 2 ? t.ylds[m * W + 1] : 0ull;
    auto bit = [&](int q) -> int { return (int)(((q < 64 ? y : yh) >> (q & 63)) & 1ull); };
    auto out = [&](int q) { return t.stage[m * t.stage_ld + q - lv.ta] + t.hbl[q - lv.ta]; };
    const bool constrained = g.n_up >= 0 && g.n_dn >= 0;
    uint64_t ahead = 0;                                        // brings the next tile's rows into L2
    if (leaf && wv == kWaves - 1 && row0 + M + m < rows) ahead = ta.x[(row0 + M + m) * W];
    const int tend = leaf ? n : lv.tb;
    int bad = sum > 0.0;
    for (int q = lv.ta + ((sub - lv.ta) & (NSUB - 1)); q < tend; q += NSUB) {
      const S o = out(q);
      const int b = bit(q);
      bool f0 = false, f1 = false;
      if (constrained) forced<W>(g, y, yh, q, spin_at(g, q), f0, f1);
      bad |= (f0 && b) || (f1 && !b);
      if (!(f0 || f1)) sum -= (double)softplus<S>(b ? -o : o);
    }
    asm volatile("" ::"v"(ahead));
    if (bad) sum = 1.0;
    if (!leaf) {
      ((double*)(st + state_units<P>(g, lv.cb) * (2 * M) * (long long)sizeof(S)))[sub * (2 * M) + half + m] = sum;
      return;
    }
    double* part = (double*)t.act;                             // in the place of the activations
    part[sub * M + m] = sum;
    lds_barrier();
    if (tid < M && m < c) {
      double v[NSUB];
#pragma unroll
      for (int i = 0; i < NSUB; ++i) v[i] = part[i * M + m];
      bad = 0;
#pragma unroll
      for (int i = 0; i < NSUB; ++i) bad |= v[i] > 0.0;
#pragma unroll
      for (int off = NSUB / 2; off >= 1; off >>= 1)
#pragma unroll
        for (int i = 0; i < off; ++i) v[i] += v[i + off];
      const double la = bad ? -INFINITY : 0.5 * v[0];
      if (g.net_kind == 1) ta.out[2 * (row0 + m)] = la;
      else ((double2*)ta.out)[row0 + m] = make_double2(la, (double)out(n + 2 * bit(n - 2) + bit(n - 1)));
    }
  };

  // The walk of a segment.  A level's tiles cover the rows up to cur[j]; its
  // next tile takes the next M nodes once they lie in rows that the level above
  // has covered, so every tile but a segment's last is full.  Node o of a level
  // has place o mod 2 M in the level's state: of the two tiles kept, a new one
  // replaces the older, which the fewer than M nodes still waiting below it
  // (all under the newer one, of M nodes) no longer need.
  long long issued = 0;
  for (long long sg = blockIdx.x; sg < nseg; sg += gridDim.x) {
    const long long s0 = sg * seg;
    const int len = (int)(rows - s0 < seg ? rows - s0 : seg);
    const uint64_t* xs = ta.x + s0 * W;
    const int last = ta.nlev - 1;
    lds_barrier();
    int lc = 0, lpar = -1;                                     // the last level's cursors, in registers
    if (thread_index() < last) {
      cur[thread_index()] = 0;                                 // rows covered
      pb[thread_index()] = -1;                                 // last node of the level above that started before cur
      tiles[thread_index()] = 0;
    }
    for (int j = 0;;) {
      if (j == last) {
        // Every row is a node, so one wave collects a tile; the others are past
        // the last use of the tile before (its partial sums' barrier).  Like
        // the levels above, with rows to be counted over all waves, five
        // barriers: 29.9 ms where this takes 28.4 (64 qubits, 400 samples).
        const int lim = __builtin_amdgcn_readfirstlane(cur[j - 1]);
        if (lc == len) break;                                  // (the levels above wait for the last one)
        const int c = lim - lc < M ? lim - lc : M;
        if (lim < len && c < M) {
          --j;
          continue;
        }
        if (wv == 0) {
          const int lane = thread_index(), r = lc + lane;
          const bool in = lane < c;
          const bool fp = in && (r == 0 || common_prefix<W>(xs, r, n) < ta.lev[j - 1].d);
          const unsigned long long bp = __ballot(fp);
          const int ip = lpar + __popcll(bp & ((2ull << lane) - 1));
          const int first = __builtin_amdgcn_readfirstlane(ip);
          if (lane < M) {                                      // a tile's empty places repeat its first node
            t.pidx[lane] = (in ? ip : first) & (2 * M - 1);
            t.put_prefix(lane, xs + (long long)(in ? r : lc) * W, n);
          }
          lpar += __popcll(bp);
        }
        lds_barrier();
        issued += ta.lev[j].flops;
        tile(j, c, 0, s0 + lc);
        lc += c;
        continue;
      }
      lds_barrier();
      const int tid = thread_index(), lane = tid & 63;
      const int c0 = __builtin_amdgcn_readfirstlane(cur[j]);
      const int lim = j > 0 ? __builtin_amdgcn_readfirstlane(cur[j - 1]) : len;
      // Nodes start at rows that differ from the row before within the level's
      // positions; a node's parent is the last node of the level above to start.
      const int dn = ta.lev[j].d, dp = j > 0 ? ta.lev[j - 1].d : 0;
      int cnt = 0, par = __builtin_amdgcn_readfirstlane(pb[j]), buf = 0;
      for (int b0 = c0; b0 < lim && cnt <= M; b0 += kThreads) {
        const int r = b0 + tid;
        const bool in = r < lim;
        const int cp = in && r > 0 ? common_prefix<W>(xs, r, n) : 0;
        const bool fn = in && cp < dn, fp = in && cp < dp;
        const unsigned long long bn = __ballot(fn), bp = __ballot(fp);
        const unsigned long long below = (1ull << lane) - 1;
        if (lane == 0) {
          wcnt[buf * 2 * kWaves + wv] = __popcll(bn);
          wcnt[buf * 2 * kWaves + kWaves + wv] = __popcll(bp);
        }
        lds_barrier();
        int at = cnt + __popcll(bn & below), ip = par + __popcll(bp & below) + (fp ? 1 : 0);
        int tn = 0, tp = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          const int a = wcnt[buf * 2 * kWaves + w], b = wcnt[buf * 2 * kWaves + kWaves + w];
          if (w < wv) {
            at += a;
            ip += b;
          }
          tn += a;
          tp += b;
        }
        if (fn && at < M) {
          t.pidx[at] = ip & (2 * M - 1);
          t.put_prefix(at, xs + (long long)r * W, n);
        }
        if (fn && at == M) {
          nxt[0] = r;
          nxt[1] = ip - (fp ? 1 : 0);
        }
        cnt += __builtin_amdgcn_readfirstlane(tn);
        par += __builtin_amdgcn_readfirstlane(tp);
        buf ^= 1;
      }
      lds_barrier();
      if (cnt < M && lim < len) {                              // the level above has to go on first
        --j;
        continue;
      }
      const int c = cnt < M ? cnt : M;
      const int half = (__builtin_amdgcn_readfirstlane(tiles[j]) & 1) * M;
      const int ce = cnt > M ? __builtin_amdgcn_readfirstlane(nxt[0]) : lim;
      const int np = cnt > M ? __builtin_amdgcn_readfirstlane(nxt[1]) : par;
      lds_barrier();
      if (tid >= c && tid < M) {                               // a tile's empty places repeat its first node
        t.pidx[tid] = t.pidx[0];
#pragma unroll
        for (int w = 0; w < W; ++w) t.ylds[tid * W + w] = t.ylds[w];
      }
      if (tid == 0) {
        cur[j] = ce;
        pb[j] = np;
        tiles[j] += 1;
      }
      lds_barrier();
      issued += ta.lev[j].flops;
      tile(j, c, half, s0 + c0);
      __syncthreads();                                         // the states are written
      ++j;
    }
  }
  if (ta.prof_slot && threadIdx.x == 0)
    atomicAdd((unsigned long long*)ta.issued, (unsigned long long)issued);
}

// One step of the sampler's walk: every entry of the buffer is a node whose
// prefix is its bits so far.  Within a level, step t takes the entry's state at
// the level's first unit (place anc[i]: the entry it descends from when the
// state was written) and evaluates only the own units that position t reads:
// cond[i] = (logit at t, forcing code).  Once the level's positions are drawn,
// a step with t < 0 writes the states of the next level.  Row by row every
// step evaluated the whole network: 94 us a step at 60 qubits, 1024 units and
// 16,384 entries; now 24 us, the three steps that write states among them.
template <int P, int W, int MB>
__global__ __launch_bounds__(kThreads, 4) void sample_units(Geom g, StepArgs sa) {
  using S = typename Kind<P>::S;
  constexpr int M = Shape<P, MB>::M;
  extern __shared__ uint4 smem[];
  const TileLds<P, W, MB> t(smem, sa.own_max, 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const S* biases = (const S*)((const char*)sa.packed + g.bias_byte);
  const Weights wb = weights(g, sa.packed);
  const long long rows = *sa.d_u < sa.umax ? *sa.d_u : sa.umax;
  for (long long r0 = (long long)blockIdx.x * M; r0 < rows; r0 += (long long)gridDim.x * M) {
    lds_barrier();
    const int tid = thread_index();
    const long long row = r0 + tid < rows ? r0 + tid : r0;
    if (tid < M) {
      t.put_prefix(tid, sa.x + row * W, g.n);
      t.pidx[tid] = sa.ca == 0 ? 0 : sa.anc ? sa.anc[row] : (int)row;
    }
    lds_barrier();
    tile_units<P, W, MB>(g, t, wb, biases, sa.ksplit, wv,
                     TileJob{sa.ca, sa.cb, sa.eb, sa.t < 0 ? 0 : sa.t, sa.t < 0 ? 0 : sa.t + 1, sa.t < 0, sa.pst,
                             sa.nodes, sa.st, sa.nodes, (int)r0},
                     [] {});
    if (sa.t >= 0 && tid < M && r0 + tid < rows) {
      const uint64_t y = t.ylds[tid * W], yh = W == 2 ? t.ylds[tid * W + 1] : 0ull;
      bool f0 = false, f1 = false;
      if (g.n_up >= 0 && g.n_dn >= 0) forced<W>(g, y, yh, sa.t, spin_at(g, sa.t), f0, f1);
      sa.cond[row] = make_double2((double)(t.stage[tid] + t.hbl[0]), f1 ? 2.0 : f0 ? 1.0 : 0.0);
    }
  }
}

// ------------------------------------------------------------------ host side
namespace {

template <int P>
bool plan_levels(const Geom& g, TreePlan& t) {
  using T = Kind<P>;
  constexpr int M = 2 * T::TB;
  const int most = T::SLOTS * kWaves * T::RB / 2;        // own blocks a workgroup can hold
  t.args = TreeArgs{};
  t.rows = M;
  TreeArgs& a = t.args;
  int ca = 0, ta = 0;
  long long bytes = 0;
  // Cuts in 32nds of the units.  A last level of a quarter of 1024 units keeps
  // two workgroups' activations in a CU's LDS.  At 512 units and fewer the
  // phases around the layers weigh more than the products saved, and a last
  // level of 7/16 is faster (40 qubits, 512 units: 52 ms a step, 61 ms with the
  // cuts of the wide network, 69 ms with one cut at half).
  const int wide[] = {8, 16, 24}, narrow[] = {10, 18};
  const bool is_wide = g.h > 512;
  for (int k = 0; k < (is_wide ? 3 : 2); ++k) {
    const int want = g.NB * (is_wide ? wide[k] : narrow[k]) / 32;
    if (want == 0) continue;
    int d = 1;
    while (d < g.n - 1 && prefix_of_class(g, d) < want * T::TB) ++d;
    const int units = prefix_of_class(g, d);
    const int cb = units / T::TB, eb = (units + T::TB - 1) / T::TB;
    if (cb <= ca || cb >= g.NB || d >= g.n - 1) continue;
    TreeLevel& lv = a.lev[a.nlev++];
    lv.ca = ca;
    lv.cb = cb;
    lv.eb = eb;
    lv.d = d;
    lv.ta = ta;
    int tb = ta;
    while (tb < d && prefix_of_class(g, tb) <= cb * T::TB) ++tb;
    lv.tb = tb;
    lv.st = bytes;
    bytes += state_units<P>(g, cb) * 2 * M * (long long)sizeof(typename T::S) + 2LL * M * sum_lanes(P) * 8;
    ca = cb;
    ta = tb;
  }
  if (a.nlev == 0) return false;
  TreeLevel& lf = a.lev[a.nlev++];
  lf = TreeLevel{ca, g.NB, g.NB, g.n, ta, g.n, 0, 0};
  int rows = 0;
  for (int k = 0; k < a.nlev; ++k) {
    // MFMA flops of a tile: fragments of layer 1 (exact inputs: one product fewer), the hidden layers and the head
    TreeLevel& lv = a.lev[k];
    const int KB = T::TB / T::KSTEP, ka = lv.ca * KB;
    const bool leaf = k + 1 == a.nlev;
    long long in = 0, own = 0, head = 0;
    for (int b = lv.ca; b < lv.eb; ++b) {
      in += g.ks1[b];
      own += std::min(g.ksh[b], lv.eb * KB) - ka;
    }
    for (int nb = 0; nb < g.NHB; ++nb)
      if (!leaf || T::TB * (nb + 1) > lv.ta) head += std::max(0, (leaf ? g.kso[nb] : std::min(g.kso[nb], lv.cb * KB)) - ka);
    const int mult = g.prec == P_BF16X3 ? 3 : g.prec == P_BF16W ? 2 : 1;
    lv.flops = 2LL * T::TB * T::KSTEP * M *
               (std::max(1, mult - 1) * in + mult * ((g.L - 1) * (own + (long long)(g.NB - lv.cb) * (lv.cb - lv.ca) * KB) + head));
    a.own_max = std::max(a.own_max, a.lev[k].eb - a.lev[k].ca);
    rows = std::max(rows, (k + 1 < a.nlev ? a.lev[k].tb : g.n + 4) - a.lev[k].ta);
  }
  if (a.own_max > most || a.own_max * T::TB > kThreads) return false;
  // the input fragments of layer 1 share the activations' place
  const int kb = T::TB / T::KSTEP;
  a.own_max = std::max(a.own_max, (g.ks1[g.NB - 1] + T::PL * kb - 1) / (T::PL * kb));
  a.stage_ld = rows | 1;
  a.scratch_wg = (bytes + 255) & ~255LL;
  t.lds = (size_t)T::PL * a.own_max * (T::TB / T::KSTEP) * 2 * 1024 +
          ((size_t)M * a.stage_ld + (size_t)a.own_max * T::TB + a.stage_ld + 1) * sizeof(typename T::S);
  t.lds += (size_t)M * 8 * g.words + (size_t)M * 4 + (16 + 4 * kWaves) * 4;
  return t.lds <= 160 * 1024;
}

// The LDS opt-in of a kernel, once per device ordinal, safe across threads.
template <typename K>
void lds_opt_in(K kern, std::atomic<unsigned long long>& done) {
  int dev = 0;
  (void)hipGetDevice(&dev);
  const unsigned long long bit = 1ull << (dev & 63);
  if (!(done.load(std::memory_order_acquire) & bit)) {
    (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    done.fetch_or(bit, std::memory_order_release);
  }
}

template <int P, int W>
void launch_w(const Geom& g, const TreePlan& t, const TreeArgs& a, int grid, hipStream_t s) {
  static std::atomic<unsigned long long> done{0};
  lds_opt_in(tree_forward<P, W>, done);
  hipLaunchKernelGGL((tree_forward<P, W>), dim3((unsigned)grid), dim3(kThreads), t.lds, s, g, a);
}

template <int P, int W, int MB>
void launch_step_w(const Geom& g, const TreePlan& t, const StepArgs& a, int grid, hipStream_t s) {
  static std::atomic<unsigned long long> done{0};
  lds_opt_in(sample_units<P, W, MB>, done);
  hipLaunchKernelGGL((sample_units<P, W, MB>), dim3((unsigned)grid), dim3(kThreads), t.lds, s, g, a);
}

// Tiles of one row block up to as many entries as tiles of two would give each
// CU one of: 23.8 us a step at 60 qubits, 1024 units and 16,384 entries, in whole
// tiles 25.5; at 24 qubits, 256 units, FP32 and 1,000 entries 9.6, 10.9.
template <int P>
void launch_step(const Geom& g, const TreePlan& t, const StepArgs& a, int cus, hipStream_t s) {
  const bool half = a.umax <= (long long)t.rows * cus;
  const long long rows = half ? t.rows / 2 : t.rows;
  const int grid = (int)std::min<long long>((a.umax + rows - 1) / rows, 2LL * cus);
  if (half) {
    if (g.words == 2) launch_step_w<P, 2, 1>(g, t, a, grid, s);
    else launch_step_w<P, 1, 1>(g, t, a, grid, s);
  } else {
    if (g.words == 2) launch_step_w<P, 2, 2>(g, t, a, grid, s);
    else launch_step_w<P, 1, 2>(g, t, a, grid, s);
  }
}

}  // namespace

size_t sample_state_bytes(const Geom& g, int cb, long long entries) {
  const long long units = g.prec == P_F64 ? state_units<P_F64>(g, cb) : state_units<P_F32>(g, cb);
  return (size_t)units * (size_t)entries * (g.prec == P_F64 ? 8 : 4);
}

void launch_sample_units(const Geom& g, const TreePlan& t, const StepArgs& sa, int cu_count, hipStream_t s) {
  StepArgs a = sa;
  a.own_max = t.args.own_max;
  const int cus = std::max(cu_count, 1);
  switch (g.prec) {
    case P_BF16: return launch_step<P_BF16>(g, t, a, cus, s);
    case P_BF16X3: return launch_step<P_BF16X3>(g, t, a, cus, s);
    case P_BF16W: return launch_step<P_BF16W>(g, t, a, cus, s);
    case P_F32: return launch_step<P_F32>(g, t, a, cus, s);
    case P_F64: return launch_step<P_F64>(g, t, a, cus, s);
  }
}

bool tree_plan(const Geom& g, TreePlan& t) {
  if (g.order_kind != 2 || g.net_kind == 2) return false;
  switch (g.prec) {
    case P_BF16: return plan_levels<P_BF16>(g, t);
    case P_BF16X3: return plan_levels<P_BF16X3>(g, t);
    case P_BF16W: return plan_levels<P_BF16W>(g, t);
    case P_F32: return plan_levels<P_F32>(g, t);
    case P_F64: return plan_levels<P_F64>(g, t);
  }
  return false;
}

int tree_head_ksplit(const Geom& g, int waves, int rows) {
  const int size = g.prec == P_F64 ? 8 : 4, mb = rows / g.TB;
  const int sp = (64 * g.words + 4 + g.TB - 1) / g.TB * g.TB + 1;
  auto floor2 = [](int v) { return v >= 8 ? 8 : v >= 4 ? 4 : v >= 2 ? 2 : 1; };
  const int fit = floor2(131072 / (rows * sp * size)), want = mb >= waves ? 1 : floor2(waves / mb);
  const int npairs = g.NHB * mb;
  return npairs >= waves ? 1 : std::min(std::min(want, fit), waves / npairs);
}

void launch_tree_forward(const Geom& g, const TreePlan& t, int ksplit, const void* packed, const uint64_t* x,
                         long long rows_bound, const long long* d_count, double* out, long long* prof_slot,
                         long long* issued, void* scratch, int grid, hipStream_t s) {
  if (rows_bound <= 0 || grid <= 0) return;
  TreeArgs a = t.args;
  a.packed = packed;
  a.x = x;
  a.d_count = d_count;
  a.bound = rows_bound;
  a.out = out;
  a.prof_slot = prof_slot;
  a.issued = issued;
  a.scratch = (char*)scratch;
  a.ksplit = ksplit;
  grid = (int)std::min<long long>(grid, (rows_bound + t.rows - 1) / t.rows);
#define NQS_TREE(P)                                                     \
  if (g.prec == P) {                                                    \
    if (g.words == 2) launch_w<P, 2>(g, t, a, grid, s);                 \
    else launch_w<P, 1>(g, t, a, grid, s);                              \
    return;                                                             \
  }
  NQS_TREE(P_BF16) NQS_TREE(P_BF16X3) NQS_TREE(P_BF16W) NQS_TREE(P_F32) NQS_TREE(P_F64)
#undef NQS_TREE
}

}  // namespace nqs
