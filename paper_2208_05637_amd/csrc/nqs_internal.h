// Internal declarations shared by the host side (nqs_capi.cpp) and the HIP
// kernels.  Nothing here is part of the C ABI.
#pragma once
#include "net.h"

namespace nqs {

// Tensor of the Hamiltonian on the device.  Masks and bit strings take
// `words` 64-bit words each (word w = qubits 64w .. 64w+63).
struct HamDev {
  const uint64_t* gx;
  const long long* goff;
  const uint64_t* tz;
  const double* tre;
  const double* tim;   // nullptr when every folded coefficient is real
  int G;
  int gfirst;          // 1 if group 0 is the empty flip
  int filter;          // spin-sector filter on
  int words;           // 1 or 2
  long long max_gterms;  // terms of the largest group past the empty flip
  // structured matrix elements (tables != 0): sub-groups soff[g] .. soff[g+1],
  // off-flip masks su[s][words], table of sub-group s at stab[s], 2^m entries
  // indexed by the bits of x at fpos[4g .. 4g+3] (-1 unused)
  int tables;
  const long long* soff;
  const uint64_t* su;
  const long long* stab;
  const double* tabre;
  const double* tabim;   // nullptr when every folded coefficient is real
  const int8_t* fpos;
};

// ---- launchers (kernels_*.hip) -------------------------------------------
void launch_fill_u32(void* p, unsigned v, long long count, hipStream_t s);
void launch_fill_u64(void* p, unsigned long long v, long long count, hipStream_t s);

void launch_diag(const HamDev& H, const uint64_t* x, long long S, double* diag, hipStream_t s);
void launch_count(const HamDev& H, const uint64_t* x, long long S, int R, int gper, int* cnt,
                  hipStream_t s);
// exclusive scan; tmp holds scan_tiles(n) + 1 values
long long scan_tiles(long long n);
void launch_scan(const int* cnt, long long n, long long* off, long long* tmp, hipStream_t s);
// one wave per sample and range, its lanes on the range's groups (else one thread)
bool write_by_wave(bool tables, long long max_gterms);
void launch_write(const HamDev& H, const uint64_t* x, long long S, int R, int gper,
                  const long long* off, long long cap, uint64_t* xe, double* he, int* esample,
                  int hstride, unsigned* err, hipStream_t s);

// Distinct keys of xe[0 .. min(*d_count, cap)) (`words` 64-bit words each)
// into xu, eu[e] = index of entry e's key in xu, *d_nu = their number, through
// `table`: HT records of kHashRecBytes (HT a power of two above the count).
// first_order: xu in the order of the keys' first entries (first: int[cap],
// rank: i64[cap + 1], rank_tmp: dedup_rank_tmp_elems(cap)); otherwise in the
// order their inserts filled the table (first, rank, rank_tmp unused).
// all_ones_key: one-word keys may be the all-ones word (64 qubits), so the
// table takes slot words instead of keys.  After the call the table maps each
// key (one-word keys below 64 qubits) to its index in xu.
constexpr size_t kHashRecBytes = 16;
long long dedup_rank_tmp_elems(long long cap);
void launch_dedup(const uint64_t* xe, int words, bool all_ones_key, const long long* d_count, long long cap,
                  void* table, long long HT, bool first_order, int* eu, uint64_t* xu, long long* d_nu, int* first,
                  long long* rank, long long* rank_tmp, unsigned* err, hipStream_t s);
// Look-back of a chunk's distinct configurations xu[0 .. *d_nu) into the
// previous chunk's one-word table (ptable, after that chunk's launch_dedup):
// src[u] = the previous index or -1; the new ones compacted in order into
// xnew, *d_nnew = their number, rank[u] = the position of a new one.
// isnew: int[cap], rank: i64[cap + 1], rank_tmp: dedup_rank_tmp_elems(cap).
void launch_lookback(const uint64_t* xu, const long long* d_nu, long long cap, const void* ptable, long long HT,
                     int* src, int* isnew, long long* rank, long long* rank_tmp, uint64_t* xnew, long long* d_nnew,
                     hipStream_t s);
// lp[u] = lp_prev[src[u]] where src[u] >= 0, else lp_new[rank[u]] (pairs of
// doubles), u < *d_nu.
void launch_lookback_gather(const long long* d_nu, long long cap, const int* src, const long long* rank,
                            const double* lp_prev, const double* lp_new, double* lp, hipStream_t s);

// Distinct configurations of the entries by their place in a map of all 2^n
// configurations (one-word strings, n <= kSectorQubits), from a base address
// on: log psi of `configs` configurations (the sector's number), their list in
// ascending order, a record per 64 places (its set bits and the number of the
// first), the tiles' numbers, tile[tiles] the number of all of them, the map.
constexpr int kSectorQubits = 28;
constexpr int kSectorTile = 4096;
struct alignas(16) SectorRec {
  unsigned long long bits;
  int base, pad;
};
struct SectorBytes {
  long long tiles;
  size_t xu, rec, tile, seen, total;
};
SectorBytes sector_bytes(int n, long long configs);
void launch_sector_index(const uint64_t* xe, const long long* d_count, long long cap, int n, int n_up, int n_dn,
                         const SectorBytes& b, void* base, hipStream_t s);

// partials holds reduce_partials_elems(S) doubles; log psi of entry e is
// lpe[eu[e]] with eu, lpe[number of xe[e]] with rec (a sector index), else lpe[e]
long long reduce_partials_elems(long long S);
void launch_reduce(long long S, int R, const long long* off, long long cap, const double* diag,
                   const double* he, int hstride, const int* eu, const uint64_t* xe, const SectorRec* rec, int n,
                   const double* lpe, const double* lps, double* eloc, double* partials, unsigned* err, hipStream_t s);
void launch_energy(const double* eloc, const double* w, long long B, double* energy,
                   unsigned* err, hipStream_t s);

// Prefix-shared forward of the connected configurations (kernels_tree.hip).
// Level of the prefix tree: the units of blocks [ca, eb) are evaluated for
// each distinct prefix of d positions, the chains of blocks [cb, NB) run over
// blocks [ca, cb) into the state at byte st of the workgroup's scratch, and the
// log-sigmoids of positions [ta, tb) are complete.  The last level's nodes are
// the rows.
constexpr int kTreeLevels = 4;
struct TreeLevel {
  int ca, cb, eb, d, ta, tb;
  long long st;
  long long flops;   // MFMA flops of one tile
};
struct TreeArgs {
  const void* packed;
  const uint64_t* x;
  const long long* d_count;   // nullable: then rows = bound
  long long bound;
  double* out;
  long long* prof_slot;       // nullable: receives the row count
  long long* issued;          // with prof_slot: receives the MFMA flops on top
  char* scratch;              // scratch_wg bytes per workgroup
  long long scratch_wg;
  int nlev, ksplit, own_max, stage_ld;
  TreeLevel lev[kTreeLevels];
};
struct TreePlan {
  TreeArgs args;
  size_t lds;
  int rows;   // nodes of a tile
};
// Levels of the network's tree; false where it has none (a sampling order the
// enumeration does not walk depth first, the dense phase network, a network of
// too few blocks).
bool tree_plan(const Geom& g, TreePlan& t);
// Rows of a segment where `grid` workgroups of tiles of M rows share `rows`.
// Segments repeat the upper levels' first tiles, so there are few: one per
// workgroup up to 3,072 rows each, else about four, of at most 16,384 rows
// (four from 1,024 rows on: a training step at 24 qubits, 1,668 rows per
// workgroup, 1.86 ms instead of 1.73; at 28 qubits, 2,100 rows, 2.37 of 2.25).
__host__ __device__ inline long long tree_segment(long long rows, long long grid, int M) {
  long long seg = (rows + grid - 1) / grid;
  if (seg > 3072) seg = (seg + 3) / 4;
  seg = seg > 16384 ? 16384 : (seg + M - 1) / M * M;
  return seg < M ? M : seg;
}
// k slices of the row-by-row forward's head with that workgroup shape.
int tree_head_ksplit(const Geom& g, int waves, int rows);
// log psi (modulus only for net_kind 1) of rows [0, min(*d_count, rows_bound))
// of x, equal to launch_forward's logits with that shape's head slices.
void launch_tree_forward(const Geom& g, const TreePlan& t, int ksplit, const void* packed, const uint64_t* x,
                         long long rows_bound, const long long* d_count, double* out, long long* prof_slot,
                         long long* issued, void* scratch, int grid, hipStream_t s);

// One step of the sampler's walk over its entries (kernels_tree.hip): units of
// blocks [ca, eb) from the states pst of the units before ca; t >= 0: cond[i] =
// (logit at position t, code 0 free, 1 forced to 0, 2 forced to 1); t < 0: the
// states of blocks [cb, NB) into st.  nodes: places per unit of the states.
struct StepArgs {
  const void* packed;
  const uint64_t* x;
  const long long* d_u;
  long long umax;
  const int* anc;      // place of entry i's state in pst; nullptr: i
  const char* pst;
  char* st;
  double2* cond;
  unsigned nodes;
  int t, ca, cb, eb, ksplit, own_max;
};
size_t sample_state_bytes(const Geom& g, int cb, long long entries);
void launch_sample_units(const Geom& g, const TreePlan& t, const StepArgs& sa, int cu_count, hipStream_t s);

// backward: recompute the sample forward on S samples and accumulate the
// gradient into grad (f64, flat parameter layout).  scratch holds
// backward_scratch_elems(g, S) elements of the path's backward type
// (double for the FP64 path, float otherwise); part: room bytes for the sums
// of blocks of samples (any size: with less room fewer blocks run at once).
long long backward_scratch_elems(const Geom& g, long long S);
void launch_backward(const Geom& g, const void* wm, const uint64_t* x, long long S,
                     const double* eloc, const double* w, const double* energy, void* scratch,
                     double* grad, void* part, size_t room, hipStream_t s);

// Sampler buffers (kernels_sample.hip); capacity umax entries, children 2 umax.
struct SampleBufs {
  uint64_t* x;       // [umax] configurations, in buffer order
  long long* cnt;    // [umax] draws
  double* cond;      // [umax][2] conditional logit and forcing code
  uint64_t* kx;      // [2 umax] children
  long long* kc;     // [2 umax]
  int* eq;           // [2 umax] tie flags
  int* keep;         // [2 umax]
  long long* eqoff;  // [2 umax + 1]
  long long* koff;   // [2 umax + 1]
  long long* stmp;   // scan_tiles(2 umax) + 1
  long long* sel;    // [2] threshold, quota
  long long* d_u;    // entries in the buffer
  long long* d_nk;   // children
  int words;         // 64-bit words per configuration (x and kx hold `words` words each)
};
void launch_sample_init(uint64_t* x, int words, long long* cnt, long long n_draws, long long* d_u, hipStream_t s);
// Children of the buffer's entries, and the new buffer of at most umax of them.
// anc_in (nullptr: i), anc_out: a number per entry that its children inherit;
// kept up to kFoldEntries entries.  Beyond, the whole network is evaluated at
// every position and the elimination takes ten launches: each workgroup of the
// one-launch elimination reads all counts, which grows with the square of the
// buffer, and the walk's states take up to 16 KB an entry (1024 units, L = 4: 2 GiB at
// the limit).  Drawing at 60 qubits with that network: 16.6 ms at 131,072 entries,
// 61 ms at one more; at 24 qubits, 256 units, FP32: 2.1 and 7.9 ms.
constexpr long long kFoldEntries = 131072;
void launch_sample_step(const SampleBufs& b, long long umax, int t, int q, uint64_t seed, const int* anc_in,
                        int* anc_out, hipStream_t s);
void launch_sample_finish(const SampleBufs& b, long long umax, uint64_t* ox, double* ow, long long* on,
                          hipStream_t s);

// Adam coefficients, formed on the host: bc1 = 1 - b1^t, bc2 = 1 - b2^t.
struct AdamCoef {
  double lr, b1, b2, one_m_b1, one_m_b2, bc1, bc2, eps;
};
void launch_adam(long long n, float* p, const double* g, double* m, double* v, const AdamCoef& k, int cu_count,
                 hipStream_t s);

}  // namespace nqs
