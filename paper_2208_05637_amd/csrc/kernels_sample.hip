// Unique-sample autoregressive sampler (Sec. 4, Sampling).
//
// A buffer of distinct configurations with occurrence counts starts as one
// configuration (all qubits 0) carrying every draw.  At sampling position t
// (qubit q = order[t]) each entry is doubled into children with x_q = 0 and
// x_q = 1, its draws are split between them by a binomial draw with the
// network's conditional P(x_q = 1 | earlier positions) (forced to 0 or 1 by
// the Hamming-weight modifier), empty children are dropped and, beyond the
// buffer capacity, the children with the fewest draws are eliminated (ties
// broken by buffer order).  The buffer order is kept sorted by the bits in
// sampling order: children with x_q = 0 come first, each group in parent
// order.
//
// Random numbers: Philox4x64 with 10 rounds (Salmon et al., SC 2011),
// counter (parent configuration's low word, t, its high word, j) for blocks
// j = 0, 1, ..., key (seed, 0), so a draw does not depend on the entry's place
// in the buffer.  Binomial Bin(c, p), exact: with q = min(p, 1 - p),
// inversion of the distribution function summed from k = 0 when c q < 32,
// else Hormann's BTRS rejection method; reflected when p > 1/2.  The arithmetic is written in
// a fixed operation order without contraction into fused multiply-adds, so a
// host implementation of the same definition draws the same counts.
#include "nqs_internal.h"

#pragma clang fp contract(off)

namespace nqs {

__device__ __forceinline__ void philox4x64_10(uint64_t (&c)[4], uint64_t k0, uint64_t k1) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += W0;
      k1 += W1;
    }
    const uint64_t hi0 = __umul64hi(M0, c[0]), lo0 = M0 * c[0];
    const uint64_t hi1 = __umul64hi(M1, c[2]), lo1 = M1 * c[2];
    const uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

__device__ __forceinline__ double uniform53(uint64_t w) {
  return (double)(w >> 11) * (1.0 / 9007199254740992.0);
}

// The uniforms of one draw: the four words of Philox block j = 0, 1, ... of
// the counter (c0, c1, c2, j), in order.
struct Uniforms {
  uint64_t c0, c1, c2, key, j;
  uint64_t w[4];
  int used;
  __device__ Uniforms(uint64_t a, uint64_t b, uint64_t c, uint64_t k) : c0(a), c1(b), c2(c), key(k), j(0), used(4) {}
  __device__ double next() {
    if (used == 4) {
      uint64_t blk[4] = {c0, c1, c2, j};
      philox4x64_10(blk, key, 0ull);
#pragma unroll
      for (int i = 0; i < 4; ++i) w[i] = blk[i];
      used = 0;
      ++j;
    }
    const int i = used++;
    return uniform53(i == 0 ? w[0] : (i == 1 ? w[1] : (i == 2 ? w[2] : w[3])));
  }
};

// fc(k) = log(k!) - [(k + 1/2) log(k + 1) - (k + 1) + log(2 pi) / 2] for integer-valued k >= 0.
__device__ double stirling_corr(double k) {
  if (k < 16.0) return lgamma(k + 1.0) - ((k + 0.5) * log(k + 1.0) - (k + 1.0) + 0.5 * log(2.0 * 3.141592653589793));
  const double x = k + 1.0;
  const double x2 = x * x;
  return (1.0 / 12.0 - (1.0 / 360.0 - (1.0 / 1260.0 - (1.0 / 1680.0) / x2) / x2) / x2) / x;
}

// log(a! / b!) for a >= b >= 0, as d log(b+1) + (a + 1/2) log1p(d/(b+1)) - d + fc(a) - fc(b), d = a - b:
// its rounding stays at the size of the result next to 10^12.
__device__ double log_fact_ratio(long long a, long long b) {
  const long long d = a - b;
  if (d == 0) return 0.0;
  const double dd = (double)d, ad = (double)a, bd = (double)b;
  return dd * log(bd + 1.0) + (ad + 0.5) * log1p(dd / (bd + 1.0)) - dd + stirling_corr(ad) - stirling_corr(bd);
}

constexpr int kMaxAttempts = 4096;

// Bin(n, p), p <= 1/2, n p >= 32: Hormann's BTRS (transformed rejection with
// squeeze; J. Statist. Comput. Simul. 46, 1993), each attempt on the next two
// uniforms; the acceptance test compares log V with log f(k)/f(m) at the mode
// m.  Attempts are capped (each accepts with probability above 0.75); at the
// cap the draw is the mode.
__device__ long long binomial_btrs(long long n, double p, Uniforms& uni) {
  const double nd = (double)n;
  const double q = 1.0 - p;
  const double spq = sqrt(nd * p * q);
  const double b = 1.15 + 2.53 * spq;
  const double a = -0.0873 + 0.0248 * b + 0.01 * p;
  const double c = nd * p + 0.5;
  const double vr = 0.92 - 4.2 / b;
  const double alpha = (2.83 + 5.1 / b) * spq;
  const double lpq = log(p / q);
  const long long m = (long long)floor((nd + 1.0) * p);
  for (int it = 0; it < kMaxAttempts; ++it) {
    const double u = uni.next() - 0.5;
    double v = uni.next();
    const double us = 0.5 - fabs(u);
    const double kf = floor(us > 0.0 ? (2.0 * a / us + b) * u + c : -1.0);   // us = 0 only at u = -1/2
    if (us >= 0.07 && v <= vr) return (long long)kf;
    if (kf < 0.0 || kf > nd) continue;
    const long long k = (long long)kf;
    v = v * alpha / (a / (us * us) + b);
    // log f(k)/f(m) = log(m!/k!) + log((n-m)!/(n-k)!) + (k - m) log(p/q)
    const double lr = k >= m ? -log_fact_ratio(k, m) + log_fact_ratio(n - m, n - k)
                             : log_fact_ratio(m, k) - log_fact_ratio(n - k, n - m);
    if (v == 0.0 || log(v) <= lr + (double)(k - m) * lpq) return k;
  }
  return m;
}

__device__ long long binomial_draw(long long c, double p, Uniforms& uni) {
  if (c == 0 || !(p > 0.0)) return 0;
  if (!(p < 1.0)) return c;
  const bool flip = p > 0.5;
  const double q = flip ? 1.0 - p : p;
  const double cd = (double)c;
  long long k;
  if (cd * q < 32.0) {
    const double u1 = uni.next();
    const double r = q / (1.0 - q);
    double pk = exp(cd * log1p(-q));
    double F = pk;
    k = 0;
    // terms past the underflowing tail are 0: stopping there bounds the
    // search even when u1 lies above the rounded total of the distribution
    while (u1 > F && k < c && pk > 0.0) {
      pk *= r * (double)(c - k) / (double)(k + 1);
      k += 1;
      F += pk;
    }
  } else {
    k = binomial_btrs(c, q, uni);
  }
  return flip ? c - k : k;
}

__global__ void sample_init_kernel(uint64_t* x, int words, long long* cnt, long long n_draws, long long* d_u) {
  for (int w = 0; w < words; ++w) x[w] = 0;
  cnt[0] = n_draws;
  *d_u = 1;
}

// Children of entry i: (x, c - k) at i and (x | 1 << q, k) at U + i.  The
// counter of the draw is (x's low word, t, x's high word, 0).
template <int W>
__global__ void sample_split_kernel(const uint64_t* __restrict__ x, const long long* __restrict__ cnt,
                                    const double2* __restrict__ cond, const long long* __restrict__ d_u,
                                    long long umax, int t, int q, uint64_t seed, uint64_t* __restrict__ kx,
                                    long long* __restrict__ kc, long long* __restrict__ d_nk) {
  const long long U = *d_u;
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *d_nk = 2 * U;
  if (i >= U || i >= umax) return;
  const double2 cd = cond[i];
  const int code = (int)cd.y;
  const double p1 = code == 1 ? 0.0 : (code == 2 ? 1.0 : 1.0 / (1.0 + exp(-cd.x)));
  uint64_t xi[W];
#pragma unroll
  for (int k = 0; k < W; ++k) xi[k] = x[i * W + k];
  Uniforms uni(xi[0], (uint64_t)t, W == 2 ? xi[W - 1] : 0ull, seed);
  const long long c = cnt[i];
  const long long k1 = binomial_draw(c, p1, uni);
#pragma unroll
  for (int k = 0; k < W; ++k) {
    kx[i * W + k] = xi[k];
    kx[(U + i) * W + k] = xi[k] | ((q >> 6) == k ? (1ull << (q & 63)) : 0ull);
  }
  kc[i] = c - k1;
  kc[U + i] = k1;
}

constexpr int kSelThreads = 1024;

__device__ long long block_count_ge(const long long* kc, long long nk, long long v, long long* sh) {
  long long n = 0;
  for (long long i = threadIdx.x; i < nk; i += kSelThreads) n += kc[i] >= v ? 1 : 0;
  for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = n;
  __syncthreads();
  long long tot = 0;
  for (int k = 0; k < kSelThreads / 64; ++k) tot += sh[k];
  __syncthreads();
  return tot;
}

// Threshold of the elimination: sel[0] = tau, sel[1] = quota.  Children with
// more than tau draws are kept, and the first `quota` (in buffer order) with
// exactly tau; tau = 0 keeps every non-empty child.
__global__ __launch_bounds__(kSelThreads) void sample_select_kernel(const long long* __restrict__ kc,
                                                                   const long long* __restrict__ d_nk,
                                                                   long long umax, long long* __restrict__ sel) {
  __shared__ long long sh[kSelThreads / 64];
  const long long nk = *d_nk;
  long long tau = 0, quota = 0;
  if (block_count_ge(kc, nk, 1, sh) > umax) {
    long long mx = 0;
    for (long long i = threadIdx.x; i < nk; i += kSelThreads) mx = kc[i] > mx ? kc[i] : mx;
    for (int o = 32; o >= 1; o >>= 1) {
      const long long v = __shfl_xor(mx, o);
      mx = v > mx ? v : mx;
    }
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = 0;
    for (int k = 0; k < kSelThreads / 64; ++k) mx = sh[k] > mx ? sh[k] : mx;
    __syncthreads();
    // largest tau with at least umax children of >= tau draws
    long long lo = 1, hi = mx + 1;
    while (hi - lo > 1) {
      const long long mid = lo + (hi - lo) / 2;
      if (block_count_ge(kc, nk, mid, sh) >= umax) lo = mid;
      else hi = mid;
    }
    tau = lo;
    quota = umax - block_count_ge(kc, nk, tau + 1, sh);
  }
  if (threadIdx.x == 0) {
    sel[0] = tau;
    sel[1] = quota;
  }
}

__global__ void sample_tie_flags(const long long* __restrict__ kc, const long long* __restrict__ d_nk,
                                 const long long* __restrict__ sel, long long n2, int* __restrict__ eq) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n2) return;
  const long long tau = sel[0];
  eq[i] = (i < *d_nk && tau > 0 && kc[i] == tau) ? 1 : 0;
}

__global__ void sample_keep_flags(const long long* __restrict__ kc, const long long* __restrict__ d_nk,
                                  const long long* __restrict__ sel, const long long* __restrict__ eqoff,
                                  long long n2, int* __restrict__ keep) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n2) return;
  const long long tau = sel[0], quota = sel[1];
  bool k = false;
  if (i < *d_nk) {
    const long long c = kc[i];
    k = c > tau || (tau > 0 && c == tau && eqoff[i] < quota);
  }
  keep[i] = k ? 1 : 0;
}

template <int W>
__global__ void sample_compact_kernel(const uint64_t* __restrict__ kx, const long long* __restrict__ kc,
                                      const int* __restrict__ keep, const long long* __restrict__ koff,
                                      long long n2, uint64_t* __restrict__ x, long long* __restrict__ cnt,
                                      long long* __restrict__ d_u) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *d_u = koff[n2];
  if (i >= n2 || !keep[i]) return;
  const long long d = koff[i];
#pragma unroll
  for (int k = 0; k < W; ++k) x[d * W + k] = kx[i * W + k];
  cnt[d] = kc[i];
}

template <int W>
__global__ void sample_finish_kernel(const uint64_t* __restrict__ x, const long long* __restrict__ cnt,
                                     const long long* __restrict__ d_u, long long umax, uint64_t* __restrict__ ox,
                                     double* __restrict__ ow, long long* __restrict__ on) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long U = *d_u;
  if (i == 0) *on = U;
  if (i >= U || i >= umax) return;
#pragma unroll
  for (int k = 0; k < W; ++k) ox[i * W + k] = x[i * W + k];
  ow[i] = (double)cnt[i];
}

// The step's elimination and compaction in one workgroup, for small buffers
// (below kShareEntries entries): the same threshold, quota and order as the kernels
// above.  Ten launches of a few microseconds each and 40 passes of the
// bisection over the counts took 130 us a step at 16,384 entries (60 us at
// 1,000); this takes 30 us (8 us): two to four passes over the counts and one
// over the children, each bound by the latency of one CU's loads.
//
// Threshold: the counts are binned by their magnitude and next five bits (exact
// below 64), the bin that holds the umax-th largest count is found from the
// top, and the remaining bits of that bin's counts are binned 11 at a time.
constexpr int kFoldBins = 2048;
__device__ __forceinline__ int fold_bin(unsigned long long v) {
  const int e = 63 - __clzll((long long)v);
  return e < 5 ? (int)v : (e - 4) * 32 + (int)((v >> (e - 5)) & 31);
}

// From the top, the bin in which the running count reaches `want` (>= 1): bin
// and the count above it.  Every thread gets both.
__device__ void fold_find(const unsigned* hist, long long want, long long* sh, int& bin, long long& above) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // thread t holds bins 2047 - 2t and 2046 - 2t
  const long long a = hist[kFoldBins - 1 - 2 * t], b = hist[kFoldBins - 2 - 2 * t];
  long long run = a + b;
  for (int o = 1; o < 64; o <<= 1) {
    const long long u = __shfl_up(run, o);
    if (lane >= o) run += u;
  }
  if (lane == 63) sh[w] = run;
  __syncthreads();
  for (int k = 0; k < w; ++k) run += sh[k];
  const long long before = run - a - b;
  if (before < want && run >= want) {
    const bool first = before + a >= want;
    sh[16] = kFoldBins - 1 - 2 * t - (first ? 0 : 1);
    sh[17] = first ? before : before + a;
  }
  __syncthreads();
  bin = (int)sh[16];
  above = sh[17];
  __syncthreads();
}

template <int W>
__global__ __launch_bounds__(kSelThreads) void sample_fold_kernel(const uint64_t* __restrict__ kx,
                                                                 const long long* __restrict__ kc, long long umax,
                                                                 uint64_t* __restrict__ x, long long* __restrict__ cnt,
                                                                 const int* __restrict__ anc_in,
                                                                 int* __restrict__ anc_out, long long* d_u) {
  __shared__ unsigned hist[kFoldBins];
  __shared__ long long sh[18];
  __shared__ int ngt[kSelThreads / 64], neq[kSelThreads / 64];
  static_assert(kFoldBins == 2 * kSelThreads, "two bins per thread");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int U = (int)*d_u, nk = 2 * U;
  // each wave takes a run of children, 64 at a time in order
  const int per = ((nk + kSelThreads - 1) / kSelThreads) * 64;
  const int i0 = wv * per, i1 = i0 + per < nk ? i0 + per : nk;
  constexpr int B = 8;                           // groups of 64 in flight: the loads' latency is most of a pass
  auto load = [&](long long (&v)[B], int j) {
#pragma unroll
    for (int k = 0; k < B; ++k) v[k] = j + 64 * k < i1 ? kc[min(j + 64 * k + lane, nk - 1)] : 0;
#pragma unroll
    for (int k = 0; k < B; ++k) v[k] = j + 64 * k + lane < i1 ? v[k] : 0;
  };
  // fn(count) for the wave's children in order, 64 lanes at once; past the run's end the count is 0
  auto each = [&](auto fn) {
    for (int j = i0; j < i1; j += 64 * B) {
      long long v[B];
      load(v, j);
#pragma unroll
      for (int k = 0; k < B; ++k)
        if (j + 64 * k < i1) fn(v[k]);
    }
  };
  auto clear = [&]() {
    hist[tid] = 0;
    hist[tid + kSelThreads] = 0;
    __syncthreads();
  };
  clear();
  each([&](long long v) {
    if (v > 0) atomicAdd(&hist[fold_bin((unsigned long long)v)], 1u);
  });
  __syncthreads();
  long long nz = 0;
  {
    long long v = (long long)hist[tid] + hist[tid + kSelThreads];
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) sh[wv] = v;
    __syncthreads();
    for (int k = 0; k < kSelThreads / 64; ++k) nz += sh[k];
    __syncthreads();
  }
  long long tau = 0, quota = 0;
  if (nz > umax) {
    int bin;
    long long above, need = umax;
    fold_find(hist, need, sh, bin, above);
    need -= above;
    // the bin's counts: [lo, lo + 2^shift)
    int shift = bin < 32 ? 0 : bin / 32 - 1;
    unsigned long long lo = bin < 32 ? (unsigned long long)bin : (unsigned long long)(32 + bin % 32) << shift;
    while (shift > 0) {
      const int r = shift < 11 ? shift : 11;
      clear();
      each([&](long long v) {
        const unsigned long long d = (unsigned long long)v - lo;
        if ((d >> shift) == 0) atomicAdd(&hist[d >> (shift - r)], 1u);
      });
      __syncthreads();
      fold_find(hist, need, sh, bin, above);
      need -= above;
      shift -= r;
      lo += (unsigned long long)bin << shift;
    }
    tau = (long long)lo;
    quota = need;
  }
  int gt = 0, eq = 0;
  each([&](long long v) {
    gt += __popcll(__ballot(v > tau));
    eq += __popcll(__ballot(tau > 0 && v == tau));
  });
  if (lane == 0) {
    ngt[wv] = gt;
    neq[wv] = eq;
  }
  __syncthreads();
  int before_gt = 0, rank = 0;
  for (int k = 0; k < wv; ++k) {
    before_gt += ngt[k];
    rank += neq[k];
  }
  const int q = (int)quota;
  int dst = before_gt + (rank < q ? rank : q);
  const unsigned long long below = (1ull << lane) - 1;
  for (int j = i0; j < i1; j += 64 * B) {
    long long v[B];
    uint64_t xv[B][W];
    int an[B];
    load(v, j);
#pragma unroll
    for (int k = 0; k < B; ++k) {
      if (j + 64 * k >= i1) break;
      const int i = min(j + 64 * k + lane, nk - 1), parent = i < U ? i : i - U;
#pragma unroll
      for (int w = 0; w < W; ++w) xv[k][w] = kx[(long long)i * W + w];
      an[k] = anc_in ? anc_in[parent] : parent;
    }
#pragma unroll
    for (int k = 0; k < B; ++k) {
      if (j + 64 * k >= i1) break;
      const bool tie = tau > 0 && v[k] == tau;
      const unsigned long long be = __ballot(tie);
      const bool keep = v[k] > tau || (tie && rank + __popcll(be & below) < q);
      const unsigned long long bk = __ballot(keep);
      if (keep) {
        const int d = dst + __popcll(bk & below);
#pragma unroll
        for (int w = 0; w < W; ++w) x[(long long)d * W + w] = xv[k][w];
        cnt[d] = v[k];
        if (anc_out) anc_out[d] = an[k];
      }
      rank += __popcll(be);
      dst += __popcll(bk);
    }
  }
  if (tid == 0) *d_u = nz < umax ? nz : umax;
}

// The same on many workgroups, for buffers of kShareEntries entries and more.
// Each workgroup bins all counts and finds the bin with the umax-th largest;
// on a second reading the counts in that bin go to a list in LDS, which is
// binned further for the threshold, and those above it among the children
// before its own give its place in the buffer.  That all workgroups do the same
// costs less than passing it on (binned by the splitting kernel's lanes with
// global atomics: 51 us more there).  16,384 entries at 60 qubits: 19 us a step
// where one workgroup took 30 (24 qubits, 256 units, a whole call: 1.27 ms of
// 1.73 at 40,000 entries, 0.92 of 0.91 at 4,096, 0.93 of 0.87 at 2,048).  A bin
// of more counts than the list holds (a flat distribution) is binned from memory.
constexpr int kShareEntries = 4096;
constexpr int kShareList = 2048;

template <int W>
__global__ __launch_bounds__(kSelThreads) void sample_share_kernel(
    const uint64_t* __restrict__ kx, const long long* __restrict__ kc, const long long* __restrict__ d_nk,
    long long umax, uint64_t* __restrict__ x, long long* __restrict__ cnt, const int* __restrict__ anc_in,
    int* __restrict__ anc_out, long long* __restrict__ d_u) {
  constexpr int COPIES = 4;                      // of the histogram, by lane: fewer lanes meet in a bin
  __shared__ unsigned hist[kFoldBins * COPIES];
  __shared__ long long sh[18];
  __shared__ int wa[kSelThreads / 64], wb[kSelThreads / 64], listed;
  __shared__ unsigned long long lv[kShareList];
  __shared__ int li[kShareList];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int nk = (int)*d_nk, U = nk / 2, i0 = blockIdx.x * kSelThreads;
  if (i0 >= nk) return;
  for (int k = tid; k < kFoldBins * COPIES; k += kSelThreads) hist[k] = 0;
  if (tid == 0) listed = 0;
  __syncthreads();
  constexpr int B = 16;
  // fn(count, child) of children [0, to), the loads of B in flight
  auto each = [&](int to, auto fn) {
    for (int j = tid; j < to; j += B * kSelThreads) {
      long long v[B];
#pragma unroll
      for (int k = 0; k < B; ++k) v[k] = kc[min(j + k * kSelThreads, nk - 1)];
#pragma unroll
      for (int k = 0; k < B; ++k)
        if (j + k * kSelThreads < to) fn((unsigned long long)v[k], j + k * kSelThreads);
    }
  };
  each(nk, [&](unsigned long long v, int) {
    if (v > 0) atomicAdd(&hist[fold_bin(v) * COPIES + lane % COPIES], 1u);
  });
  __syncthreads();
  {
    unsigned a = 0, b = 0;
    for (int k = 0; k < COPIES; ++k) {
      a += hist[tid * COPIES + k];
      b += hist[(tid + kSelThreads) * COPIES + k];
    }
    __syncthreads();
    hist[tid] = a;
    hist[tid + kSelThreads] = b;
  }
  __syncthreads();
  auto block_sum = [&](int v, int* part) {
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) part[wv] = v;
    __syncthreads();
    int tot = 0;
    for (int k = 0; k < kSelThreads / 64; ++k) tot += part[k];
    return tot;
  };
  const long long nz = block_sum((int)(hist[tid] + hist[tid + kSelThreads]), wa);
  // counts of [lo, lo + 2^shift) straddle the threshold; without elimination lo = 0 and all counts are above
  unsigned long long lo = 0;
  int shift = 0, bin;
  long long above, need = 0;
  if (nz > umax) {
    need = umax;
    fold_find(hist, need, sh, bin, above);
    need -= above;
    shift = bin < 32 ? 0 : bin / 32 - 1;
    lo = bin < 32 ? (unsigned long long)bin : (unsigned long long)(32 + bin % 32) << shift;
  }
  int gt = 0, eq = 0;                            // among the children before this workgroup's
  const int end = shift > 0 ? nk : i0;
  each(end, [&](unsigned long long v, int i) {
    if (v < lo) return;
    if (((v - lo) >> shift) != 0) {
      gt += i < i0 ? 1 : 0;
    } else if (shift > 0) {
      const int at = atomicAdd(&listed, 1);
      if (at < kShareList) {
        lv[at] = v;
        li[at] = i;
      }
    } else {
      eq += 1;                                   // (lo > 0: exactly the threshold; lo = 0: an empty child)
    }
  });
  __syncthreads();
  const int m = listed;
  // fn(count, child) of the bin's counts
  auto members = [&](auto fn) {
    if (m <= kShareList) {
      for (int k = tid; k < m; k += kSelThreads) fn(lv[k], li[k]);
    } else {
      each(nk, fn);
    }
  };
  const unsigned long long blo = lo;
  const int bshift = shift;
  while (shift > 0) {
    const int r = shift < 11 ? shift : 11;
    hist[tid] = 0;
    hist[tid + kSelThreads] = 0;
    __syncthreads();
    members([&](unsigned long long v, int) {
      const unsigned long long d = v - lo;
      if (v >= lo && (d >> shift) == 0) atomicAdd(&hist[d >> (shift - r)], 1u);
    });
    __syncthreads();
    fold_find(hist, need, sh, bin, above);
    need -= above;
    shift -= r;
    lo += (unsigned long long)bin << shift;
  }
  const long long tau = (long long)lo;
  if (bshift > 0)
    members([&](unsigned long long v, int i) {
      if (i < i0 && v >= blo && ((v - blo) >> bshift) == 0) {
        gt += v > lo ? 1 : 0;
        eq += v == lo ? 1 : 0;
      }
    });
  if (tau == 0) eq = 0;
  const int gt0 = block_sum(gt, wa), eq0 = block_sum(eq, wb), q = (int)need;
  __syncthreads();
  // this workgroup's children, one per thread
  const int i = i0 + tid;
  const long long v = i < nk ? kc[i] : 0;
  const bool tie = tau > 0 && v == tau;
  const unsigned long long be = __ballot(tie), below = (1ull << lane) - 1;
  if (lane == 0) wa[wv] = __popcll(be);
  __syncthreads();
  int rank = eq0 + __popcll(be & below);
  for (int k = 0; k < wv; ++k) rank += wa[k];
  const bool keep = v > tau || (tie && rank < q);
  const unsigned long long bk = __ballot(keep);
  if (lane == 0) wb[wv] = __popcll(bk);
  __syncthreads();
  if (keep) {
    int d = gt0 + (eq0 < q ? eq0 : q) + __popcll(bk & below);
    for (int k = 0; k < wv; ++k) d += wb[k];
#pragma unroll
    for (int w = 0; w < W; ++w) x[(long long)d * W + w] = kx[(long long)i * W + w];
    cnt[d] = v;
    const int parent = i < U ? i : i - U;
    if (anc_out) anc_out[d] = anc_in ? anc_in[parent] : parent;
  }
  if (blockIdx.x == 0 && tid == 0) *d_u = nz < umax ? nz : umax;
}

static unsigned blocks_for(long long n, int t) { return (unsigned)((n + t - 1) / t); }

void launch_sample_init(uint64_t* x, int words, long long* cnt, long long n_draws, long long* d_u, hipStream_t s) {
  hipLaunchKernelGGL(sample_init_kernel, dim3(1), dim3(1), 0, s, x, words, cnt, n_draws, d_u);
}

void launch_sample_step(const SampleBufs& b, long long umax, int t, int q, uint64_t seed, const int* anc_in,
                        int* anc_out, hipStream_t s) {
  const long long n2 = 2 * umax;
  auto split = b.words == 2 ? sample_split_kernel<2> : sample_split_kernel<1>;
  // one wave per workgroup: lanes of a wave differ in how long they draw, and
  // more workgroups spread over more CUs (17 -> 15 us at 16,384 entries)
  hipLaunchKernelGGL(split, dim3(blocks_for(umax, 64)), dim3(64), 0, s, b.x, b.cnt,
                     (const double2*)b.cond, b.d_u, umax, t, q, seed, b.kx, b.kc, b.d_nk);
  if (umax >= kShareEntries && umax <= kFoldEntries) {
    auto share = b.words == 2 ? sample_share_kernel<2> : sample_share_kernel<1>;
    hipLaunchKernelGGL(share, dim3(blocks_for(n2, kSelThreads)), dim3(kSelThreads), 0, s, b.kx, b.kc, b.d_nk, umax,
                       b.x, b.cnt, anc_in, anc_out, b.d_u);
    return;
  }
  if (umax < kShareEntries) {
    auto fold = b.words == 2 ? sample_fold_kernel<2> : sample_fold_kernel<1>;
    hipLaunchKernelGGL(fold, dim3(1), dim3(kSelThreads), 0, s, b.kx, b.kc, umax, b.x, b.cnt, anc_in, anc_out, b.d_u);
    return;
  }
  hipLaunchKernelGGL(sample_select_kernel, dim3(1), dim3(kSelThreads), 0, s, b.kc, b.d_nk, umax, b.sel);
  hipLaunchKernelGGL(sample_tie_flags, dim3(blocks_for(n2, 256)), dim3(256), 0, s, b.kc, b.d_nk, b.sel, n2, b.eq);
  launch_scan(b.eq, n2, b.eqoff, b.stmp, s);
  hipLaunchKernelGGL(sample_keep_flags, dim3(blocks_for(n2, 256)), dim3(256), 0, s, b.kc, b.d_nk, b.sel,
                     b.eqoff, n2, b.keep);
  launch_scan(b.keep, n2, b.koff, b.stmp, s);
  auto compact = b.words == 2 ? sample_compact_kernel<2> : sample_compact_kernel<1>;
  hipLaunchKernelGGL(compact, dim3(blocks_for(n2, 256)), dim3(256), 0, s, b.kx, b.kc, b.keep,
                     b.koff, n2, b.x, b.cnt, b.d_u);
}

void launch_sample_finish(const SampleBufs& b, long long umax, uint64_t* ox, double* ow, long long* on,
                          hipStream_t s) {
  auto finish = b.words == 2 ? sample_finish_kernel<2> : sample_finish_kernel<1>;
  hipLaunchKernelGGL(finish, dim3(blocks_for(umax, 256)), dim3(256), 0, s, b.x, b.cnt, b.d_u,
                     umax, ox, ow, on);
}

}  // namespace nqs
