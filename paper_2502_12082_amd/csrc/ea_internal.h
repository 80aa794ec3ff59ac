// ea_internal.h -- launch interface between the C ABI (ea_api.hip) and the
// kernel translation units.  Host-side only; no torch, no exceptions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ea {

// Largest sequence length the kernels accept (the solver keeps one byte per
// (wave, key block) of mask state in LDS).
constexpr int MAX_SEQLEN = 131072;
constexpr int MAX_KEY_BLOCKS = MAX_SEQLEN / 64;

// Which specialisation of the per-element map: gamma = 1/(alpha-1) in
// {1, 2, 4} run without transcendentals; 0 means general alpha.
int gamma_kind(float alpha);

// One cached score of a later fill of the solver's lists: the raw score
// s = <q_i, k_j> (the solver forms x - tau from it exactly as in a streamed
// evaluation) and the key j.
struct alignas(8) CandEntry {
  float s;
  int32_t j;  // key index; its key block is j / 64
};

// Workgroup geometry (rows and threads per workgroup) of the solver.  Each row
// has two candidate lists (one per half of every key block), of `cap` entries
// each.
constexpr int SOLVE_ROWS = 256;
constexpr int SOLVE_THREADS = 256;

// The solver caches quads: the four raw scores of four
// consecutive keys 4 m .. 4 m + 3 that one lane holds for one row (16 bytes),
// with m as a 16-bit key (2 bytes, in an array of their own).  Its first
// evaluation copies the scores above the bracket's lower end into lists of
// single scores (4 bytes, and their key blocks, 2 bytes).  A slot holds
// `cap` quads and `cap` singles in each of the 2 * SOLVE_THREADS lists of a
// workgroup.
constexpr size_t SOLVE_QUAD_BYTES = 16 + 2;
constexpr size_t SOLVE_SINGLE_BYTES = 4 + 2;
constexpr size_t solve_slot_bytes(int cap) {
  return (size_t)cap * 2 * SOLVE_THREADS * (SOLVE_QUAD_BYTES + SOLVE_SINGLE_BYTES);
}
static_assert(MAX_SEQLEN / 4 <= 65536, "a quad's key fits 16 bits");

// Element lists: the nonzero probabilities of every row of a 64-row query
// block, written by the solver (or, in the no-mask mode's backward, by
// collect_kernel) where they are few, and read by the forward and backward
// instead of recomputing the scores of whole blocks.
// Each row has two lists of up to LIST_CAP entries (the keys that each half
// of the solver's wave held for it): z = [x - tau]_+ and the 16-bit key, entry
// e of list id = 64 * half + row at index LIST_IDS * e + id.  One record per
// query block, sized for the most it can hold (the host cannot know the counts
// without waiting for the solver): 37248 bytes, 582 a row.
constexpr int LIST_CAP = 48;
constexpr int LIST_IDS = 2 * 64;
constexpr int LIST_ENTRIES = LIST_CAP * LIST_IDS;  // at most, per query block
constexpr int LIST_MAX_SEQLEN = 65536;             // keys fit 16 bits
struct ListBlock {
  float z[LIST_ENTRIES];
  uint16_t key[LIST_ENTRIES];
  uint8_t count[LIST_IDS];
  float tau[64];  // the thresholds the z belong to
};
static_assert(sizeof(ListBlock) % 128 == 0, "records keep their alignment");
// What a block's lists serve, by its entries per listed key block (64 x 64
// scores): beyond these limits the matrix products of whole blocks are faster
// than a gather per entry and the solver's stores of them (bf16 d64, us, with
// the lists against without: B8 H12 n1024 at 76 entries per block solver and
// forward 155 against 182, dQ 47 against 59; at 97 197 against 210 and 58
// against 59; at 55 dK/dV with the sort 95 against 108; B8 H4 n1169 at 107
// solver and forward 169 against 166.  B64 H16 n128, at 512: 34 against 33, 42
// against 28, 103 against 42).  fp32 products take 16
// times as long, but a listed entry twice the bytes and a store the same: four
// and six times the limits (B8 H16 n512 d64, 136 per block: forward 31 against
// 124, dQ 41 against 127).
// Among many key blocks a few entries are always listed for dK/dV (the first
// rows of a causal head), since one block that is not makes the whole head
// take both ways; the forward and dQ of such a block are a step or two of
// products (B1 H16 n4096 d128 causal alpha 1.25, whose first blocks hold up to
// 1000 entries a key block: dQ 131 us without lists, 141 with).
// (An array of their own beside the records: kernels read one of many blocks.)
enum ListUse { LIST_NONE = 0, LIST_FWD = 1, LIST_DQ = 2, LIST_DKDV = 4 };  // bits
constexpr int LIST_MOST = 100, LIST_MOST_F32 = 600;  // entries per key block, for any use
#if defined(__HIPCC__)
__host__ __device__ inline int list_few(int T) { return 32 * T < 1024 ? 32 * T : 1024; }
__host__ __device__ inline int list_use(int entries, int blocks, int T, bool f32) {
  const int per = f32 ? 4 * blocks : blocks;
  if (entries > LIST_ENTRIES) return LIST_NONE;
  if (entries <= 64 * per) return LIST_FWD | LIST_DQ | LIST_DKDV;
  const int few = entries <= list_few(T) ? LIST_DKDV : LIST_NONE;
  return entries <= (f32 ? LIST_MOST_F32 : LIST_MOST) * blocks ? few | LIST_FWD | LIST_DQ : few;
}
#endif

struct TauArgs {
  const void* q;
  const void* k;
  float* tau;         // [BH, n]
  uint8_t* mask;      // [BH, T, T], or null (the no-mask mode: no tables either)
  int32_t* stats;     // [2, BH, T] K passes and evaluations for each 64-row query block, or null
  void* cand;         // candidate cache: one slot per workgroup, or null
  int cap;            // quads per list
  int slots;          // cache slots (workgroup b of a launch uses slot b)
  int tile0;          // first tile of this launch (workgroup b solves tile tile0 + b)
  int BH, n, T;
  float c;            // (alpha - 1) * scale
  float alpha, gamma;
  int causal, max_iter;
  float tol;
  int gk;             // gamma_kind(alpha)
  // fp32 inputs, general alpha: tau is refined in fp64 and written as
  // tau + tau_lo ([BH, n]); c64, g64 are (alpha - 1) * scale and 1/(alpha - 1)
  // in fp64 from the same fp32 parameters
  float* tau_lo;
  double c64, g64;
  // the row tables of the mask (Q_i of every query block), written with it
  int32_t* q_count;   // [BH, T]
  int32_t* q_index;   // [BH, T, T]
  ListBlock* lists;   // [BH * T] (n <= LIST_MAX_SEQLEN), or null
  int32_t* use;       // [BH * T] ListUse: 0, or the lists hold every nonzero probability
};

struct FwdArgs {
  const void* q;
  const void* k;
  const void* v;
  void* o;                // [BH, n, D] input dtype
  float* o2;              // [BH, n, D] fp32, train only
  const float* tau;
  const int32_t* q_count;
  const int32_t* q_index;
  int BH, n, T;
  float c, gamma;
  int causal;
  int gk;
  const float* tau_lo;  // fp32 inputs, general alpha: low part of tau (or null: 0)
  double c64, g64;
  // the column tables (K_j of every key block), built by extra workgroups of
  // the same launch from the mask
  const uint8_t* mask;  // [BH, T, T]
  int32_t* k_count;     // [BH, T]
  int32_t* k_index;     // [BH, T, T]
  const ListBlock* lists;  // [BH * T], or null
  const int32_t* use;      // as in TauArgs
};

// The element lists of a query block in the backward, sorted by key block
// into the call's workspace: entry p of bucket J at off[J] + p (off: [T + 1]
// per query block), with its row and key within their blocks (row * 64 + key).
struct Buckets {
  int32_t* used;   // [BH * T]: whether the block's lists serve dQ, and its buckets dK and dV
  int32_t* heads;  // [BH]: whether any block of the head has buckets
  uint16_t* off;   // [BH * T, T + 1]
  float* z;        // [BH * T, LIST_ENTRIES]
  uint16_t* code;  // [BH * T, LIST_ENTRIES]
};

struct BwdArgs {
  const void* q;
  const void* k;
  const void* v;
  const void* dout;
  const float* tau;
  const float* delta;     // [BH, n]
  const int32_t* q_count;
  const int32_t* q_index;
  const int32_t* k_count;
  const int32_t* k_index;
  float *dq, *dk, *dv;
  int BH, n, T;
  float c, gamma, scale;
  int causal;
  int gk;
  const float* tau_lo;  // fp32 inputs, general alpha: low part of tau (or null: 0)
  double c64, g64;
  const ListBlock* lists;  // [BH * T], or null; then also
  Buckets buckets;
};

struct DeltaArgs {
  const void* dout;
  const float* o2;
  float* delta;
  int64_t rows;
  // with element lists: their buckets are written too
  const ListBlock* lists;  // [BH * T], or null
  const int32_t* use;      // as in TauArgs
  const float* tau;
  Buckets buckets;
  int BH, n, T;
};

// The element lists of given thresholds (no-mask mode's backward).
struct CollectArgs {
  const void* q;
  const void* k;
  const float* tau;
  const float* tau_lo;  // as in BwdArgs
  ListBlock* lists;
  int32_t* use;  // as in TauArgs
  int32_t* est;  // scratch, at most [BH * T]: entries found in a sample of query blocks
  int BH, n, T;
  float c;
  int causal, gk;
  double c64;
};

// Row-wise alpha-entmax of a materialized [rows, n] score matrix.
struct RowsArgs {
  const void* s;      // [rows, n] scores, input dtype
  float* p;           // [rows, n] probabilities (forward output)
  float* tau;         // [rows] thresholds (forward output, backward input)
  const float* dp;    // [rows, n] gradient of p (backward input)
  float* ds;          // [rows, n] gradient of s (backward output)
  int64_t rows;
  int n;
  float c;            // (alpha - 1) * scale
  float alpha, gamma, scale, tol;
  int max_iter, gk;
};

// Largest row the row-wise kernels hold in registers.
constexpr int MAX_ROW_LEN = 32768;

// Each launcher picks the instantiation for (dtype: 0 bf16 / 1 fp32, head_dim,
// gamma kind) and returns the launch status.
// Launches `kernel` with its one argument struct and returns the launch's own
// status (not an error left behind by earlier HIP calls on this thread).
template <typename A>
inline hipError_t launch_kernel(void (*kernel)(A), dim3 grid, dim3 block, hipStream_t s, A a) {
  void* args[] = {&a};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, args, 0, s);
}

hipError_t launch_tau(const TauArgs& a, int dtype, int head_dim, hipStream_t s);
// The solver for sequences of up to SMALL_MAX_N keys, but fp32 inputs with a
// general alpha (no candidate cache, no K passes beyond the first).
constexpr int SMALL_MAX_N = 1024;
hipError_t launch_tau_small(const TauArgs& a, int dtype, int head_dim, hipStream_t s);
hipError_t launch_tau_bf16_64(const TauArgs& a, hipStream_t s);
hipError_t launch_tau_bf16_128(const TauArgs& a, hipStream_t s);
hipError_t launch_tau_f32_64(const TauArgs& a, hipStream_t s);
hipError_t launch_tau_f32_128(const TauArgs& a, hipStream_t s);
hipError_t launch_fwd(const FwdArgs& a, int dtype, int head_dim, bool train, hipStream_t s);
hipError_t launch_delta(const DeltaArgs& a, int dtype, int head_dim, hipStream_t s);
hipError_t launch_bwd_dkdv(const BwdArgs& a, int dtype, int head_dim, hipStream_t s);
// dK and dV of the listed query blocks, added to what launch_bwd_dkdv (given
// the same lists) wrote for the others.
hipError_t launch_bwd_dkdv_lists(const BwdArgs& a, int dtype, int head_dim, hipStream_t s);
// (a sample of the density, then the lists of heads that look sparse)
hipError_t launch_collect(const CollectArgs& a, int dtype, int head_dim, hipStream_t s);
hipError_t launch_bwd_dq(const BwdArgs& a, int dtype, int head_dim, hipStream_t s);
hipError_t launch_rows_fwd(const RowsArgs& a, int dtype, hipStream_t s);
hipError_t launch_rows_bwd(const RowsArgs& a, int dtype, hipStream_t s);

}  // namespace ea
