// Internal layout shared by the host planner and the gfx950 kernels.
//
// A planned problem is one contiguous device image (caller-owned workspace).
// Constraints are reordered into segments; each segment holds constraints of
// one evaluation kind and one length bucket, so a wavefront runs one code path.
#pragma once
#include <cstddef>
#include <cstdint>

namespace pcls {

// Evaluation kinds.  Every kind evaluates FE = sum_t sp_t Pr[T = t] (T = number
// of true literals under independent literals of mean y) through products of
// per-literal factors (alpha + beta * y) at a set of nodes:
//   PROD1 - one real node (sp constant except at t = 0, t = k, or alternating):
//           FE = c0 + c1 * prod_i (a + b y_i)
//   PROD2 - two real nodes (sp constant on 1..k-1):
//           FE = c0 + c1 * prod_i (1+y_i)/2 + c2 * prod_i (1-y_i)/2
//   DFT   - any spectrum: the count distribution of each lane's literals, combined across
//           a lane group at the K = KMAX+1 complex roots of unity of the length bucket
//   PMF   - sp constant outside a window of w counts at one end (thresholds,
//           at-most-one, exactly-kappa near an end), w <= 4 for k <= 8 (one lane
//           per pair) and w <= KMAX/2 of the length bucket for 17 to 48 literals (lane
//           groups): with C the number of true literals (or of false ones),
//           FE = c0 + sum_{c < w} d_c Pr[C = c], from a truncated Poisson-binomial
//           recursion and its adjoint (no complex nodes).  (Windows of 9 to 16 literals
//           are listed as PMF too and run as DFT, on one lane without nodes.)
//   CONST - sp constant: FE = c0, no literal work
//   THR   - a threshold (d constant on the window) of 9 to 64 literals whose bucket has
//           enough empty slots to pad its window to exactly KMAX/2 counts: W - w pad
//           slots hold literals whose event is certain, which shifts every count by
//           W - w.  All classes of a bucket then run the same code, and the sums over
//           the window are running sums.  (Listed as PMF up to 48 literals, as DFT above.)
enum Kind : int32_t { KIND_PROD1 = 0, KIND_PROD2 = 1, KIND_DFT = 2, KIND_PMF = 3, KIND_CONST = 4, KIND_THR = 5 };
constexpr int kPmfWindow = 4;  // counts kept by the PMF kind, one lane per pair (k <= 8)
constexpr int kPmfMaxK = 8;    // longest constraint of the one-lane PMF kind
constexpr int kThrMaxK = 64;   // longest bucket of the THR kind
constexpr int kPmfGroupMaxK = 48;  // longest constraint of the lane-group PMF kind (window <= bucket / 2)

// Length buckets of the segment kernels: literals per constraint padded to KMAX,
// processed by groups of G lanes holding J = KMAX / G literals each.
constexpr int kNumBuckets = 18;
constexpr int kBucketKmax[kNumBuckets] = {1, 2, 3, 4, 5, 6, 7, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256};
// Kernel variants, by the longest bucket they are compiled for.
constexpr int kMaxbShort = 7;                // k <= 8
constexpr int kMaxbMid = 11;                 // k <= 32
constexpr int kMaxbAll = kNumBuckets - 1;    // k <= 256
constexpr int kMaxK = 256;
// (kind, bucket) pairs of the non-constant kinds: the products and DFT have every
// bucket, PMF and THR these (the kernels' cases; LDS holds one counter a segment)
constexpr bool runs_pmf(int kmax) { return kmax <= kPmfMaxK || (kmax > 16 && kmax <= kPmfGroupMaxK); }
constexpr bool runs_thr(int kmax) { return kmax > kPmfMaxK && kmax <= kThrMaxK; }
constexpr int count_segments() {
  int count = 0;
  for (int kmax : kBucketKmax) count += 3 + runs_pmf(kmax) + runs_thr(kmax);
  return count;
}
constexpr int kMaxSegments = 72;
static_assert(count_segments() <= kMaxSegments, "a plan's segments need a counter each");
// Pad rows: problems with constraints longer than 8 literals get kPadRows extra
// rows in the on-chip state, held at x = +1 and never stepped.  A slot past a
// constraint's end (length buckets above 8) codes one of these rows, with the
// literal sign chosen so that the slot's factor is exactly 1 (its gradient
// term lands in the pad row, whose accumulator is never read).  Slot i of
// constraint q of a segment starts on pad row (q + i) mod kPadRows, so pads
// spread over banks; the planner's bank balance may then move them between
// the constraint's slots.
constexpr int kPadRows = 64;

// Lanes per (constraint, restart) pair: one lane holds up to 16 literals (register
// budget at 4 waves per SIMD); longer constraints spread over G lanes (a power of
// two) of at most 16 (12 for the buckets 24, 48, ...), products above 16 literals and
// the windows of 9 to 16 of at most 8 (6).
constexpr int lane_groups(int kmax, int per_lane = 8) {
  int g = 1;
  while (kmax > per_lane * g) g *= 2;
  return g;
}
constexpr int group_size(int kind, int kmax) {
  if (kmax <= 8) return 1;
  if (kind == KIND_THR || kind == KIND_PMF) return kmax <= 16 ? 2 : lane_groups(kmax, 16);
  return kind == KIND_DFT ? lane_groups(kmax, 16) : (kmax <= 16 ? 1 : lane_groups(kmax));
}
// What a constraint limits the tile width by (64 / width lanes are left for its
// group): the lanes of at most 8 literals, also where a kind uses fewer.
constexpr int tile_group(int kind, int kmax) {
  return kind == KIND_PROD1 || kind == KIND_PROD2 ? group_size(kind, kmax) : lane_groups(kmax);
}

// Bucket tables: which of the compiled lengths a plan uses.  Table 0 uses all of
// them; table 1 only the exact ones up to 8 and the powers of two above (fewer
// segments, more padded slots).  The autotuners choose between them.
constexpr int kNumBucketTables = 2;
inline bool bucket_in_table(int b, int table) {
  const int k = kBucketKmax[b];
  return table == 0 || k <= 8 || (k & (k - 1)) == 0;
}
inline int bucket_of(int k, int table = 0) {
  for (int b = 0; b < kNumBuckets; ++b)
    if (k <= kBucketKmax[b] && bucket_in_table(b, table)) return b;
  return -1;
}

struct Segment {
  int32_t kind;       // Kind
  int32_t bucket;     // index into kBucketKmax
  int32_t c_begin;    // first constraint (planned order)
  int32_t c_count;    // constraints in the segment
  int32_t lit_base;   // offset of the segment's transposed literal block
  int32_t par_fixed;  // product kinds: the parameters (c_par) when every constraint has these, else 0
  int32_t cls_fixed;  // >= 0 when every constraint has this class
  int32_t m_max;      // PMF: widest window over the segment
  int32_t z_off;      // DFT over a lane group: the bucket's node powers (entry of the node table)
};

// Per constraint class (type, k, param).
struct ClassRec {
  int32_t kind;
  int32_t k;
  int32_t node_off;  // DFT, PMF: offset into the node table (entries)
  int32_t window;    // PMF, THR: window w
  int32_t listed;    // kind it is counted under (pcls_info)
  int32_t sp_off;    // offset of sp[0..k] (int8) in the spectrum table
  float a, b;        // PROD1 node factor a + b y
  float c1, c2;      // PROD1 / PROD2 product weights
  float c0;          // constant term (folded into the per-problem constant on device)
  // Which counts t of true literals violate the constraint (extraction): every
  // type's spectrum alternates or changes sign at most twice, so
  // [violated] = v0 ^ (vpar & t & 1) ^ [t >= t1] ^ [t >= t2], packed as t1 in bits
  // 0..8, t2 in bits 9..17 (511 where there is none), v0 in bit 18, vpar in bit 19.
  uint32_t violated;
};

// Entry of the node table: eight floats, read by kind.
//   DFT over a lane group of J literals a lane, K = KMAX + 1: a class has the
//     KMAX/2 weights W_m = 2 chat_m (re, im; the 2 covers the conjugate node K - m),
//     and the bucket the powers z_m^1..z_m^J of every node (J real, J imaginary parts).
//   DFT on one lane: a class has sp_t - sp_k for t = 0..KMAX (0 past k).
//   PMF of k <= 8 literals: one entry {d_0, d_1, d_2, d_3, h, 0, 0, 0}, where the
//     counted event of literal i has probability 1/2 - h y_i (h = 1/2: true, -1/2:
//     false); a longer one has five: d_0..d_31 (zero past its window), h, then
//     padding.
struct NodeRec {
  float f[8];
};

// Device view of a planned problem (passed by value to kernels).
struct ProblemDev {
  int32_t n, m, L;
  int32_t n_pad;                 // pad rows after the n variables (0 or kPadRows)
  int32_t n_segments;
  int32_t n_classes;
  float f_const;                 // sum_c w_c c0_c
  const Segment* segments;
  const ClassRec* classes;
  const NodeRec* nodes;
  const int8_t* sp;              // spectra
  const int32_t* litT;           // per segment: [KMAX][c_count] literal codes: variable in bits 0..30,
                                 // bit 31 set for a negated literal; a slot past the constraint's
                                 // end codes a pad row (variable >= n)
  const int32_t* c_cls;          // per constraint class
  int32_t n_codes;               // entries of litT
  const int32_t* c_par;          // per constraint of a product kind: two bf16 values, PROD1 b and c1,
                                 // PROD2 c2 and c1 (high and low half); of a DFT one: its class's
                                 // node table entry; of a PMF one: its class; of a THR one: h and
                                 // d_0 (two bf16 values)
  const float* c_w;              // per constraint weight
  const int32_t* row_ptr;        // planned-order CSR (extract / streaming engine)
  const int32_t* lit;            // planned-order literal codes
  const uint32_t* c_viol;        // per constraint: ClassRec::violated
  int32_t const_unsat;           // violated constraints among those of constant spectrum
  int32_t unit_weights;          // all weights 1.0
  int32_t pair_terms;            // one restart a tile: one objective term a (constraint, restart) pair (set by the kernel, in a batch by the host)
  int32_t max_k;
  const int32_t* occ;            // per variable: occurrences in non-constant constraints
  const int32_t* perm;           // planned index -> caller's constraint index
};

}  // namespace pcls
