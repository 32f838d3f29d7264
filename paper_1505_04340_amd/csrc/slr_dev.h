// Device-side layout of an SLR preconditioner and the kernel launchers.
// All device vectors are FP64, column-major, in the internal DD order
// (interiors by subdomain, then the interface in C's factor order).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <cstdint>

namespace slr {

// Per-subdomain descriptor of the batched B_i solves (offsets into the
// concatenated arrays of all subdomains).
//
// Each sweep of each subdomain is packed as a level-sliced byte stream
// (built on the host, 16-byte aligned segments); lvb[l] is the byte offset
// of level l's segment (lvb[nlev] = total bytes).  For level l with L rows:
//
// Fixed width K (every row of every sweep padded to the problem's widest
// row K <= 4; padding has w = 0 and points at the row itself; levels wider
// than 64 * rec_passes(K) rows split), row records of KR = rec_width(K)
// entries:
//     idx   int32[L][KR]       [row, c_0, .., c_{K-1}, pad]  local indices
//     wts   TS[L][KR]          [sc, w_0, .., w_{K-1}, pad]   scale, weights
// Any width (pack_K == 0): a "level" is a segment of at most about kSegBytes
// (unless one task is larger), a list of tasks with a program for each of
// the kSegWaves solver waves:
//     uint16    barriers inside the segment, words of the longest program,
//               place / 16 of the flat program, its words
//     uint32    words[i][wave]   programs, then the flat one of all tasks
//     tasks     16-byte aligned, offsets / 16 from the segment's start
// A word (SegWord): bits 0-11 the task's place / 16, 12-13 its type, 14-16
// and 17-25 its shape, 26-31 the barriers to pass before it.
//   kSegEnd
//   kSegEll    14-16 log2 of the lanes per row, 17-25 nu entries per lane
//     rows  uint32[64]         local row of each lane (bit 31: not stored)
//     sc    TS[64]             row scale
//     ci    uint16[nb][64][B]  columns; B = 2 (nu <= 2) or 4, nb = ceil(nu / B)
//     w     TS[nb][64][B]      pre-divided weights
//     (lane g of a row's G lanes holds its entries g, g + G, ..; padding has
//     w = 0 and column m, one past the rows, which is zero)
//   kSegChain  14 with entries to the previous chain, 17-25 R rows
//     rows  uint16[16]         the chain's rows in solve order (the last repeated)
//     prev  uint16[16]         the previous chain's
//     w     TS[16][16]         [c][i]: weight of row c in row i
//     v     TS[16][16]         that of the previous chain's row c
//   kSegPanel  17-25 R rows
//     cols  uint16[16]         rows of a finished chain
//     rows  uint16[64]
//     w     TS[16][R]          [c][j]: weight of row c in row j
struct BlockDesc {
  int32_t m0, m;                   // interior range in the internal order
  int32_t f_nlev, f_K, f_lev, f_lvb;   // forward sweep: levels, width, levptr / lvb offsets
  int32_t b_nlev, b_K, b_lev, b_lvb;   // backward sweep
  int64_t f_data, b_data;          // byte offsets of the packed streams
  // E rows (interior rows coupled to the interface), ELL with width e_K:
  //   e_row[e_row + i] local row; e_q / e_val[e_ent + e*e_n + i] (padding: q 0, value 0)
  int32_t e_row, e_n, e_K, e_ent;
  // E^T rows (interface rows owned here), ELL with width t_K:
  //   t_q[t_row + i] interface index; t_j / t_val[t_ent + e*t_n + i] (padding: j 0, value 0)
  int32_t t_row, t_n, t_K, t_ent;
};

// Interface sweeps (C): level-scheduled CSR on the device, see slr_host.h.
// rp entries are absolute offsets into ci / w.
template <typename TS>
struct SweepArrays {
  const int32_t *lev = nullptr;    // level pointers
  const int32_t *rows = nullptr;   // level-sorted rows
  const int32_t *rp = nullptr;     // nrows+1 absolute entry offsets
  const int32_t *ci = nullptr;     // column indices
  const TS *w = nullptr;           // pre-scaled off-diagonal weights
  const TS *sc = nullptr;          // per-row scale
  const TS *w2 = nullptr;          // two-level schedules: w * sc of the dependency row
};

template <typename TS>
struct BlockArrays {
  const BlockDesc *desc = nullptr;
  const int32_t *lev = nullptr;    // level pointers of all sweeps
  const int32_t *lvb = nullptr;    // level byte offsets of all sweeps
  const uint8_t *data = nullptr;   // packed sweep streams
  const uint16_t *e_row = nullptr;
  const int32_t *e_q = nullptr;
  const TS *e_val = nullptr;
  const int32_t *t_q = nullptr;
  const uint16_t *t_j = nullptr;
  const TS *t_val = nullptr;
  // LDS position of interior row m0 + r of a block (r local): every local
  // index above (packed streams, E rows, E^T columns) is such a position;
  // null: position = local row in every block
  const uint16_t *xpos = nullptr;
  int32_t max_m = 0;
  int32_t max_lev = 0;
  int32_t max_level_bytes = 0;     // largest single level segment
  int32_t max_K = 0;               // widest packed row over all sweeps
  int32_t pack_K = 0;              // > 0: every packed row has exactly this width
};

// What one launch of the batched B kernel computes for each subdomain i
// and right-hand side column c (columns [0, nrhs)):
//   rhs   = a_f * f_i + b_y * E_i y           (prologue)
//   z     = B_i^{-1} rhs                      (forward + backward sweep in LDS)
//   u_i   = z                                 (if u != nullptr)
//   gout_q = c_g * g_q + d_t * (E^T z)_q      (epilogue, q owned by i; if gout)
// LDS bytes after the B kernel's stage that absorb the prologue's stores
// past the end of x's rows: one 16-byte slot per lane of a wave, so that
// such stores from one instruction never hit the same bank.
constexpr int kStageDummyBytes = 1024;
// Segments of sweeps of any width: solver waves, stager waves, columns from which each wave
// takes columns of its own, bytes aimed at, task types
constexpr int kSegWaves = 6, kSegStagers = 2, kSegColumns = 4, kSegHeaderBytes = 16, kSegBytes = 8192, kChainRows = 16;
constexpr int kSegEnd = 0, kSegEll = 1, kSegChain = 2, kSegPanel = 3;

// Entries of a fixed-width row record: the row plus K columns, rounded up to
// a multiple of 4 so that records are whole 16-byte vectors.
__host__ __device__ constexpr int rec_width(int K) { return (K + 1 + 3) & ~3; }

// Row passes per lane the fixed-width sweep kernel unrolls for rows of width
// K (bounded by registers); the host splits wider levels into consecutive
// sub-levels of at most 64 * rec_passes(K) rows (rows of one level are
// independent, so any split of a level is a valid schedule).
__host__ __device__ constexpr int rec_passes(int K) { return K <= 2 ? 4 : (K == 3 ? 3 : 2); }

// Most threads of a B kernel workgroup.  Sweeps of any width: the solver waves
// that their programs are laid out for and the stagers; with fewer waves each
// solver wave takes columns of its own.
__host__ __device__ constexpr int bsolve_threads(int pack_K) { return pack_K > 0 ? 1024 : 64 * (kSegWaves + kSegStagers); }

// A column of x in LDS: m values, and a zero for the padding of sweeps of any
// width.  Bytes of the R columns of a workgroup (max_m: rows of the largest).
__host__ __device__ constexpr int x_stride(int m, int pack_K) { return pack_K > 0 ? m : m + 1; }
__host__ __device__ constexpr int64_t x_bytes(int64_t value, int max_m, int pack_K, int R) {
  return (value * (pack_K > 0 ? (int64_t)max_m * R + 1 : ((int64_t)max_m + 1) * R) + 15) & ~(int64_t)15;
}

// Sweeps of any width: slots of a ring of segments in the stage.
__host__ __device__ constexpr int ring_slots(int stage_bytes, int max_segment) {
  const int slot = (max_segment + 15) & ~15, n = stage_bytes / (slot > 0 ? slot : 1);
  return n < 8 ? n : 8;
}

struct BArgs {
  const double *f = nullptr;  int64_t ldf = 0;  double a_f = 0.0;
  const double *y = nullptr;  int64_t ldy = 0;  double b_y = 0.0;
  const double *g = nullptr;  int64_t ldg = 0;  double c_g = 0.0;
  double *gout = nullptr;     int64_t ldgo = 0; double d_t = 0.0;
  double *u = nullptr;        int64_t ldu = 0;
  // idx != nullptr: f, g and u are in the caller's order, row i of the
  // internal order (interior rows, then the interface) at idx[i]; g and gidx
  // take the interface rows' part.  With yout, y is also stored there in the
  // caller's order: each subdomain an even share of the s rows.
  const int32_t *idx = nullptr, *gidx = nullptr;
  double *yout = nullptr;     // leading dimension ldu
  int32_t s = 0, p = 1;
  int32_t nrhs = 1;
  int32_t R = 1;              // right-hand sides per workgroup
  int32_t stage_bytes = 0;    // LDS staging buffer for the packed sweeps
  int32_t sweeps = 3;         // bit 0: forward sweep, bit 1: backward sweep
  // persistent launch (sched != nullptr): workgroup w takes the work items
  // sched[sched_ptr[w] .. sched_ptr[w+1]), each (column group << 16) |
  // subdomain, in that order; otherwise blockIdx.x is the subdomain and
  // blockIdx.y the column group
  const int32_t *sched = nullptr;
  const int32_t *sched_ptr = nullptr;
  // persistent with per-subdomain column counts: items are subdomain |
  // (first column << 16) | (columns << 24), each subdomain's x stored with
  // its own row count as stride, as many columns as the x region holds
  int32_t var_cols = 0;
  int32_t shared = 0;         // several workgroups a compute unit (sweeps of any width: fewer registers)
};

// Numeric refactorisation on the device: one stored coefficient (TS) at
// byte offset `off` of its array, computed from factor values V (rounded to
// TS first when TS is FP32) or from the input matrix values:
//   RF_SRC    val[a]                     (E, E^T entries)
//   RF_ONE    1
//   RF_RAW    V[a]                        (unit-L weights of L D L^T)
//   RF_RECIP  rd(1 / V[a])                (row scales)
//   RF_DIV    rd(V[a] / V[b])             (pre-divided weights)
//   RF_W2     rd(rd(V[a] / V[b]) * rd(1 / V[c]))   (two-level interface weights)
//   RF_ENT    rd(V[a] / V[b]) / rd(1 / V[b])       (entries between the blocks of a deep factor)
//   RF_ENT64  the same, stored in FP64 whatever TS is
// rd() rounds to TS, exactly as the host packing does.
enum { RF_SRC = 0, RF_ONE, RF_RAW, RF_RECIP, RF_DIV, RF_W2, RF_ENT, RF_ENT64 };
struct RfMap {
  int64_t off;
  int32_t a, b, c, op;
};

// every map of a refactorisation that is not empty in one launch; V: the
// factor of a map's values (RF_SRC reads val)
constexpr int kRfMaps = 13;
struct RfPack {
  const RfMap *map[kRfMaps] = {};
  int64_t n[kRfMaps] = {};
  const double *V[kRfMaps] = {};
  void *base[kRfMaps] = {};
  int32_t maps = 0;
};
template <typename TS>
void launch_rf_pack(const RfPack &P, const double *val, hipStream_t st);
// *flag = 1 if some val[e] != val[tr[e]] (tr: the mirror entry of each entry)
void launch_mirror_check(int64_t n, const int64_t *tr, const double *val, int *flag, hipStream_t st);
// out[e] = val[src[e]]
void launch_gather(int64_t n, const int64_t *src, const double *val, double *out, hipStream_t st);
// Block-diagonal factor without fill whose rows have at most kFactEntries
// entries off the diagonal, no two of which share a column (no products to
// subtract): the rows of a block level by level, at most kFactThreads a
// level.  Slot r holds row (rec[r].w & 0xFFFF) of its block, its entry count
// (rec[r].w >> 16), its first entry in V (rec[r].z) and the block's rows of
// its columns, 16 bits each (rec[r].x, .y); src[u * slots + r] is the matrix
// entry of its diagonal (u = 0) and of entry u - 1 (past the end: the
// diagonal's).  Block b has the levels lev[blk[b]] .. lev[blk[b + 1]].
constexpr int kFactEntries = 4, kFactThreads = 256;
struct FactBlocks {
  const int4 *rec = nullptr;
  const int32_t *src = nullptr, *blk = nullptr, *lev = nullptr;
  int32_t slots = 0, nb = 0, max_m = 0, ldl = 0;
};
void launch_fact_blocks(const FactBlocks &F, const double *val, double *V, int *err, hipStream_t st);
// IC(0) (ldl = 0) or ILDL^T(0) (ldl = 1) of the rows rows[r0 .. r1) of the
// lower CSR (rp, ci, diagonal last) whose values V hold the matrix entries
// on entry; earlier rows must be final.  *err is set to 1 on a failed pivot.
void launch_fact_level(const int64_t *rp, const int32_t *ci, double *V, const int32_t *rows, int32_t r0, int32_t r1,
                       int32_t ldl, int *err, hipStream_t st);

template <typename TS, typename TC>
void launch_bsolve(const BlockArrays<TS> &B, int32_t p, const BArgs &a, int32_t threads,
                   size_t lds_bytes, hipStream_t st);

// In-place level-scheduled sweep of one (interface) block on a global
// vector: x (ld, nrhs columns).  Deep schedules run in one workgroup per
// column; shallow ones launch once per level over the whole device.
// G > 1 (sweeps with long rows): one launch per level, G lanes per row.
template <typename TS, typename TC>
void launch_sweep(const SweepArrays<TS> &S, const int32_t *lev_host, int32_t nlev, int32_t nrows,
                  double *x, int64_t ldx, int32_t nrhs, bool one_wg, hipStream_t st, int32_t G = 1);

// Out-of-place sweep of a schedule with at most two levels, one launch.
// dv (optional, nrhs == 1): per-block partial sums of dv . y to dpart
// ((nrows + 255) / 256 blocks).
template <typename TS, typename TC>
void launch_sweep2(const SweepArrays<TS> &S, int32_t nrows, const double *x, int64_t ldx, double *y, int64_t ldy,
                   int32_t nrhs, hipStream_t st, const double *dv = nullptr, double *dpart = nullptr);

// End of Lanczos step j (k_lanczos_next: beta_j from the partials bpart,
// v_{j+1} = w / beta_j, the recorded coefficients) together with the next
// step's first sweep: tout = L^{-T} v_{j+1} by the two-level backward
// schedule S (nw2 weight entries), equal to launch_sweep2 of v_{j+1}.
template <typename TS>
void launch_lanczos_next_sweep(int64_t s, int32_t j, const double *w, double *vnext, double *sc, double *alpha,
                               double *beta, const double *bpart, int32_t rb, const double *aval,
                               const SweepArrays<TS> &S, int64_t nw2, double *tout, hipStream_t st);

// Rank-k block of eq. skt on w (s x nrhs, ld ldw), output to wout (ldo);
// U column-major s x k:
//   c = U^T w ;  c_i <- c_i * dsc_i ;  wout = rho * w + U c
template <typename TU>
void launch_lowrank(const TU *U, int64_t s, int32_t k, const double *dsc, double rho,
                    const double *w, int64_t ldw, double *wout, int64_t ldo, int32_t nrhs,
                    double *part, int32_t nblk, double *cbuf, unsigned int *counter,
                    hipStream_t st);

}  // namespace slr
