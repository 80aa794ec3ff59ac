// ea_bwd.hip -- sparse alpha-entmax attention backward.
//
// With tau from the forward, u_ij = [x_ij - tau_i]_+^(gamma-1) on the support
// (= p^(2-alpha), the sparse Jacobian Diag(u) - u u^T / |u|_1 of Sec. 3.2.2)
// and O2 saved by the forward (App. A.2):
//   delta_i = <dO_i, O2_i>                                   (App. A.2)
//   dP_ij   = <dO_i, v_j>,  dS_ij = u_ij (dP_ij - delta_i)    (App. A.2)
//   dV_j = sum_{i in K_j} P_ij^T dO_i                         (Eq. 13)
//   dK_j = scale * sum_{i in K_j} dS_ij^T q_i                 (Eq. 12)
//   dQ_i = scale * sum_{j in Q_i} dS_ij k_j                   (Eq. 11)
// split into a delta pre-kernel, a dK/dV kernel over key blocks and a dQ
// kernel over query blocks (Algorithms 4 and 5, visiting only the blocks of
// the lookup tables as in App. A.5).  `scale` appears because the entmax
// input is scale * Q K^T; no alpha factor survives the chain rule.
//
// Precision: S and dP are bf16 x bf16 products accumulated in fp32; P is
// rounded to bf16 for P^T dO; dS is fed to the MFMA as a two-term bf16 split
// (hi + lo) so dK and dQ keep ~16 mantissa bits of dS; outputs are fp32.
//
// gfx950 layout: 32 resident rows per wave in registers (K and V rows for
// dK/dV; Q and dO rows for dQ); the other side's 64-row tiles are copied by
// global_load_lds into row-major LDS tiles (two stages; three in the bf16
// d = 128 dK/dV kernel), read directly for S and dP and through transposing
// LDS reads for the permuted contractions P^T dO, dS^T Q and dS K.  The dK/dV
// work has two forms: dkdv_kernel (2 waves per key block, every column) and,
// for bf16 at d = 128, dkdv2_kernel (8 waves over two key blocks, each wave
// half of the columns, S and dP operands shared through LDS).  No atomics:
// every output row has one owner, so results are deterministic.
#include <type_traits>

#include "ea_common.h"
#include "ea_internal.h"

namespace ea {

namespace {

constexpr int BWD_NT = 128;

// ------------------------------------------------------------------ delta

template <typename E, int D>
__global__ __launch_bounds__(256) void delta_kernel(DeltaArgs a) {
  constexpr int PER = D / 16;  // 16 lanes per row
  const long long row = (long long)blockIdx.x * 16 + (threadIdx.x >> 4);
  const int sl = threadIdx.x & 15;
  float acc = 0.f;
  if (row < a.rows) {
    const E* dO = static_cast<const E*>(a.dout) + row * D + sl * PER;
    const float* o2 = a.o2 + row * D + sl * PER;
#pragma unroll
    for (int e = 0; e < PER; ++e) acc = fmaf((float)dO[e], o2[e], acc);
  }
#pragma unroll
  for (int m = 8; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
  if (row < a.rows && sl == 0) a.delta[row] = acc;
}

// ------------------------------------- element lists sorted by key block

// Lanes whose `key` (of `bits` bits) equals the calling lane's, among the
// lanes of `active`.
__device__ __forceinline__ unsigned long long same_key(int key, int bits, unsigned long long active) {
  unsigned long long m = active;
  for (int b = 0; b < bits; ++b) {
    const unsigned long long set = __ballot((key >> b) & 1);
    m &= (key >> b) & 1 ? set : ~set;
  }
  return m;
}
__device__ __forceinline__ int lanes_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

constexpr int PREP_NT = 256;
constexpr int PREP_T = LIST_MAX_SEQLEN / BLK;  // most key blocks
constexpr int PREP_STAGE = 3072;               // entries that fit the staging memory
constexpr int PREP_SMALL = 2048;               // blocks of a small grid
static_assert(PREP_SMALL <= (PREP_NT / 64) * PREP_T && PREP_SMALL >= PREP_T, "a counter per head, and a head's blocks");
// Buckets::used: the block's lists are good (for dQ), and sorted (for dK, dV)
constexpr int LISTED = 1, SORTED = 2;

// One workgroup per 64-row query block: delta of its rows, and, where the
// forward listed the block, its entries sorted by key block for the dK/dV
// kernel (a counting sort: each wave takes 32 of the 128 lists, counts its
// entries per key block, and places them after those of the waves before).
// Entries of one key block keep the order of (wave, entry, list), so the sort
// is deterministic.  The lists are used only if their thresholds are the
// residuals' (a forward that did not write lists may have filled the
// residuals again).
template <typename E, int D>
__global__ __launch_bounds__(PREP_NT) void prep_kernel(DeltaArgs a) {
  constexpr int PER = D / 16;  // 16 lanes per row
  constexpr int W = PREP_NT / 64;
  __shared__ uint32_t cursor[W][PREP_T];
  __shared__ float zs[PREP_STAGE];
  __shared__ uint16_t cs[PREP_STAGE];
  __shared__ uint32_t wsum[W];
  const int t = threadIdx.x, lane = lane_id(), w = wave_id();
  const int bh = blockIdx.x / a.T, qb = blockIdx.x % a.T;
  const size_t blk = blockIdx.x;
  const int nr = min(BLK, a.n - qb * BLK);
  const long long row0 = (long long)bh * a.n + (long long)qb * BLK;
  // uses of the head's blocks, or of every head's in a small grid (see below)
  const bool small = sizeof(E) == 2 && a.BH * a.T <= PREP_SMALL;
  const int h0 = small ? 0 : bh, heads = small ? a.BH : 1;
  int all_use[PREP_SMALL / PREP_NT];
#pragma unroll
  for (int k = 0; k < PREP_SMALL / PREP_NT; ++k) {
    const int x = t + k * PREP_NT;
    all_use[k] = x < heads * a.T ? a.use[(size_t)h0 * a.T + x] : 0;
  }
#pragma unroll
  for (int r = t >> 4; r < BLK; r += PREP_NT / 16) {
    float acc = 0.f;
    if (r < nr) {
      const E* dO = static_cast<const E*>(a.dout) + (row0 + r) * D + (t & 15) * PER;
      const float* o2 = a.o2 + (row0 + r) * D + (t & 15) * PER;
#pragma unroll
      for (int e = 0; e < PER; ++e) acc = fmaf((float)dO[e], o2[e], acc);
    }
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) acc += __shfl_xor(acc, m);
    if (r < nr && (t & 15) == 0) a.delta[row0 + r] = acc;
  }

  const ListBlock& lb = a.lists[blk];
  const int T = a.T;
  bool same = true;
  if (t < nr) same = __float_as_uint(lb.tau[t]) == __float_as_uint(a.tau[row0 + t]);
  const int use = __syncthreads_and(same) ? a.use[blk] : LIST_NONE;
  // The dK/dV work of a head is split only if at least 7 of 8 of its blocks
  // are listed: the others cost a pass of their own over every key block.  A
  // small grid takes as long as its longest workgroup, so there every head has
  // to be so.  (dK/dV and sort, with against without lists, in us: B1 H4
  // n11392 d128 causal, 537 of 712 blocks listed 689 against 459, 618 of them
  // 303 against 470; B8 H8 n3000 d64 causal, 2192 of 3008 329 against 234;
  // B4 H12 n4096 d64 causal, 2478 of 3072 319 against 306.)  fp32 products take
  // 16 times as long: three quarters of the head alone do there (step of B1 H2
  // n1984 d128 causal c = 0.6 1030 us against 1456 with the rule of bf16).
  bool split = true;
  if (use & LIST_DKDV || qb == 0) {
    uint32_t* const rest = &cursor[0][0];  // unlisted blocks of each head
    for (int h = t; h < heads; h += PREP_NT) rest[h] = 0;
    __syncthreads();
    const float per_head = 1.f / (float)T;
#pragma unroll
    for (int k = 0; k < PREP_SMALL / PREP_NT; ++k) {
      const int x = t + k * PREP_NT;  // (its head exactly: x < 2^11)
      if (x < heads * T && !(all_use[k] & LIST_DKDV)) atomicAdd(&rest[(int)(((float)x + 0.5f) * per_head)], 1u);
    }
    __syncthreads();
    for (int h = t; h < heads; h += PREP_NT) split &= (sizeof(E) == 2 ? 8 : 4) * (int)rest[h] <= T;
    split = __syncthreads_and(split);
    if (qb == 0 && t == 0) a.buckets.heads[bh] = split;
  }
  const bool sorted = (use & LIST_DKDV) && split;
  if (t == 0) a.buckets.used[blk] = (use & LIST_DQ ? LISTED : 0) | (sorted ? SORTED : 0);
  if (!sorted) return;

  const int bits = 32 - __clz(max(T - 1, 1));
  for (int x = t; x < W * T; x += PREP_NT) cursor[x / T][x % T] = 0;
  const int id = 32 * w + (lane & 31), half = lane >> 5, cnt = lb.count[id];
  int most = cnt;  // longest list of the wave
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) most = max(most, __shfl_xor(most, o));
  // Lanes below 32 take the even entries of their list, the others the odd;
  // loads in batches of eight entries per lane.
  constexpr int B = 8;
  auto keys = [&](int e0, int (&key)[B]) {
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int e = e0 + 2 * u + half;
      key[u] = e < cnt ? (int)lb.key[LIST_IDS * e + id] : -1;
    }
  };
  __syncthreads();
  for (int e0 = 0; e0 < most; e0 += 2 * B) {
    int key[B];
    keys(e0, key);
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (key[u] >= 0) atomicAdd(&cursor[w][key[u] >> 6], 1u);
  }
  __syncthreads();
  // exclusive sums in the order (key block, wave)
  uint16_t* const off = a.buckets.off + blk * (size_t)(T + 1);
  const int per = (T + PREP_NT - 1) / PREP_NT;
  uint32_t mine = 0;
  for (int k = 0; k < per; ++k) {
    const int j = t * per + k;
    if (j < T)
      for (int x = 0; x < W; ++x) mine += cursor[x][j];
  }
  uint32_t incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t v = __shfl_up(incl, o);
    if (lane >= o) incl += v;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  uint32_t start = incl - mine;
  for (int x = 0; x < w; ++x) start += wsum[x];
  const uint32_t total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  for (int k = 0; k < per; ++k) {
    const int j = t * per + k;
    if (j < T) {
      off[j] = (uint16_t)start;
      for (int x = 0; x < W; ++x) {
        const uint32_t v = cursor[x][j];
        cursor[x][j] = start;
        start += v;
      }
    }
  }
  if (t == 0) off[T] = (uint16_t)total;
  __syncthreads();
  float* const zg = a.buckets.z + blk * LIST_ENTRIES;
  uint16_t* const cg = a.buckets.code + blk * LIST_ENTRIES;
  const bool staged = total <= PREP_STAGE;
  for (int e0 = 0; e0 < most; e0 += 2 * B) {
    int key[B];
    float z[B];
    keys(e0, key);
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int e = e0 + 2 * u + half;
      z[u] = e < cnt ? lb.z[LIST_IDS * e + id] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const bool ok = key[u] >= 0;
      const unsigned long long act = __ballot(ok);
      if (act == 0ull) break;
      const int kb = key[u] >> 6;
      const unsigned long long m = same_key(kb, bits, act);
      if (ok) {
        const int rank = lanes_below(m);
        const uint32_t p = cursor[w][kb] + (uint32_t)rank;
        if (rank == __popcll(m) - 1) cursor[w][kb] = p + 1;  // (all lanes have read it by then)
        const uint16_t code = (uint16_t)((id & 63) * 64 + (key[u] & 63));
        if (staged) {
          zs[p] = z[u];
          cs[p] = code;
        } else {
          zg[p] = z[u];
          cg[p] = code;
        }
      }
    }
  }
  if (!staged) return;
  __syncthreads();
  for (uint32_t p = t; p < total; p += PREP_NT) {
    zg[p] = zs[p];
    cg[p] = cs[p];
  }
}

// ------------------------------- element lists from the thresholds alone

// The element lists of the no-mask mode's backward, which is given thresholds
// but no lists: one K pass at tau (one of the three products a block of dQ
// and dK/dV each costs otherwise), every z > 0 appended to its row's lists.
// Workgroup = 128 rows, wave = 32 rows against both halves of every key block,
// as the solver's one-group form.  A wave whose lists overflow stops scoring,
// and the workgroup stops when all have.
//
// That pass costs as much as it can gain where a block holds COL_MOST entries
// per key block (backward, us, products against lists: B1 H8 n2431 d128 at 40
// entries 181 against 192, at 20 180 against 147; B4 H21 n3136 d64 causal at
// 37 535 against 582, at 26 529 against 486), and more where rows are too long
// for their lists.  So probe_kernel first counts the entries of a sample of
// the scores, 64 rows x 128 keys of every eighth query block, and
// collect_kernel leaves a head that looks denser than that alone (about 10 us,
// where the whole pass was 115 us of 895 at B4 H21 n3136 d64 causal c = 0.5;
// with every query block sampled probe_kernel took 15 us at B1 H16 n4096 d128).
// With a general alpha the maps of the products take longer, and both limits
// are higher (B2 H3 n11674 d64 alpha 1.75 c = 0.3: 1975 against 3261 us a step).
// fp32 calls always collect: their products take 16 times as long, and the
// sample 20 us.
constexpr int COL_NT = 256;
constexpr int COL_MOST = 28;          // entries per key block (twice that with a general alpha)
constexpr int COL_SAMPLE = 4;         // sub-tiles of 32 keys, per sampled query block
constexpr int COL_EVERY = 8;          // query blocks a sampled one stands for: 4, 12, 20, ...
// entries of a block some of whose rows (40 or 56 on average) may not fit 2 x LIST_CAP
constexpr int COL_LONG = 2600, COL_LONG_GENERAL = 3600;

__host__ __device__ inline int sampled_blocks(int T) { return (T + COL_EVERY - 1) / COL_EVERY; }
__host__ __device__ inline int sampled_block(int s, int T) {
  return COL_EVERY * s + COL_EVERY / 2 < T ? COL_EVERY * s + COL_EVERY / 2 : T - 1;
}

template <typename E, int D>
__global__ __launch_bounds__(COL_NT) void probe_kernel(CollectArgs a) {
  using M = Mma<E>;
  constexpr int KS = D / M::KW;
  __shared__ int found[COL_NT / 64];
  const int lane = lane_id(), w = wave_id();
  const int n = a.n, per = sampled_blocks(a.T), bh = blockIdx.x / per;
  const int qb = sampled_block(blockIdx.x % per, a.T);
  const int q0 = qb * BLK + 32 * (w & 1), i = q0 + (lane & 31);
  const E* Q = static_cast<const E*>(a.q) + (size_t)bh * n * D;
  const E* K = static_cast<const E*>(a.k) + (size_t)bh * n * D;
  const float tau = i < n ? a.tau[(size_t)bh * n + i] : INFINITY;
  typename M::frag qf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) qf[kk] = load_row_frag_global<E, D>(Q, i, n, kk);
  // one sub-tile of each quarter of the block's keys, another one in the next block
  const int tiles = ((a.causal ? min(n, qb * BLK + BLK) : n) + 31) / 32;
  int in = 0;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int quarter = (w >> 1) + 2 * x, t0 = quarter * tiles / COL_SAMPLE;
    const int j0 = 32 * min(t0 + (5 * qb + 3 * bh) % max(tiles / COL_SAMPLE, 1), tiles - 1);
    f32x16 s = zero16();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      s = M::mma(load_row_frag_global<E, D>(K, min(j0 + (lane & 31), n - 1), n, kk), qf[kk], s);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int j = j0 + crow(r);
      in += j < n && (!a.causal || j <= i) ? in_support(relu_z(a.c, s[r], tau)) : 0;
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) in += __shfl_xor(in, o);
  if (lane == 0) found[w] = in;
  __syncthreads();
  if (threadIdx.x == 0) a.est[blockIdx.x] = found[0] + found[1] + found[2] + found[3];
}

// Whether head bh (in a small grid, which takes as long as its slowest head:
// every head) looks sparse enough to collect.  Heads of about the same density
// go the same way, by the density of all of them: some of them listed and some
// not takes longest (B4 H21 n3136 d64 causal at 28 entries a key block: 733 us
// against 565 and 575).  `sums` holds two counters per head.  Every thread of
// the workgroup.
__device__ bool looks_sparse(const CollectArgs& a, int bh, int* sums) {
  __shared__ unsigned long long all;
  const int T = a.T, per = sampled_blocks(T), t = threadIdx.x;
  const bool small = a.BH * T <= PREP_SMALL;
  const int h0 = small ? 0 : bh, heads = small ? a.BH : 1;
  for (int h = t; h < 2 * heads; h += COL_NT) sums[h] = 0;
  if (t == 0) all = 0;
  __syncthreads();
  unsigned long long mine = 0;
  for (int x = t; x < a.BH * per; x += COL_NT) {
    const int h = x / per, s = x - h * per, blocks = a.causal ? sampled_block(s, T) + 1 : T;
    const int expected = a.est[x] * blocks;  // twice the block's entries
    mine += (unsigned)expected;
    if (h >= h0 && h < h0 + heads) {
      atomicAdd(&sums[2 * (h - h0)], expected >> 6);
      if (expected > 2 * (a.gk == 0 ? COL_LONG_GENERAL : COL_LONG)) atomicAdd(&sums[2 * (h - h0) + 1], 1);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mine += __shfl_xor(mine, o);
  if (lane_id() == 0) atomicAdd(&all, mine);
  __syncthreads();
  int valid = per * T;  // key blocks of a head's sampled query blocks
  if (a.causal) {
    valid = 0;
    for (int s = 0; s < per; ++s) valid += sampled_block(s, T) + 1;
  }
  const int most = a.gk == 0 ? 2 * COL_MOST : COL_MOST;
  const int limit = (all <= 2ull * most * valid * a.BH ? 3 * most / 2 : most / 2) * (valid / 32 + 1);
  bool sparse = true;
  for (int h = t; h < heads; h += COL_NT) sparse &= sums[2 * h] <= limit && 8 * sums[2 * h + 1] <= per;
  return __syncthreads_and(sparse);
}

template <typename E, int D, int GK>
__global__ __launch_bounds__(COL_NT, sizeof(E) == 4 && D == 128 ? 1 : 3) void collect_kernel(CollectArgs a) {
  using TL = PadTile<E, D>;
  using M = Mma<E>;
  constexpr int KS = D / M::KW;
  constexpr bool PRECISE = precise_path<E, GK>();
  __shared__ __attribute__((aligned(16))) E kbuf[2][TL::ELEMS];
  __shared__ uint32_t bits[2][PREP_T / 32];  // key blocks in use, per query block
  __shared__ int entries[2];
  const int t = threadIdx.x, lane = lane_id(), w = wave_id(), half = lane >> 5;
  const int n = a.n, T = a.T;
  int bh, qt;
  head_major(blockIdx.x, a.BH, (T + 1) / 2, bh, qt);
  if (a.causal) qt = (T + 1) / 2 - 1 - qt;
  const int q0 = qt * 128 + 32 * w, i = q0 + (lane & 31), qbl = w >> 1, qb = 2 * qt + qbl;
  const bool row_ok = i < n;
  const E* Q = static_cast<const E*>(a.q) + (size_t)bh * n * D;
  const E* K = static_cast<const E*>(a.k) + (size_t)bh * n * D;
  const int last = min(n, q0 + 32) - 1;  // last row of the wave
  const int nkb = a.causal ? (min(n, qt * 128 + 128) - 1) / BLK + 1 : T;
  const float c = a.c, tau = row_ok ? a.tau[(size_t)bh * n + i] : INFINITY;
  [[maybe_unused]] const double tau64 =
      (double)tau + (PRECISE && a.tau_lo && row_ok ? (double)a.tau_lo[(size_t)bh * n + i] : 0.0);
  [[maybe_unused]] const float band = PRECISE_BAND * fmaxf(1.f, fabsf(tau));
  static_assert(sizeof(kbuf) >= 2 * PREP_SMALL * sizeof(int), "looks_sparse");
  if (sizeof(E) == 2 && !looks_sparse(a, bh, reinterpret_cast<int*>(&kbuf[0][0]))) {
    if ((w & 1) == 0 && lane == 0 && qb < T) a.use[(size_t)bh * T + qb] = LIST_NONE;
    return;
  }
  for (int x = t; x < 2 * (PREP_T / 32); x += COL_NT) (&bits[0][0])[x] = 0;
  if (t < 2) entries[t] = 0;

  typename M::frag qf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) qf[kk] = load_row_frag_global<E, D>(Q, i, n, kk);
  ListBlock* const lb = qb < T ? a.lists + ((size_t)bh * T + qb) : nullptr;
  const int row = i - qb * BLK, id = 64 * half + row;
  int cnt = 0;
  bool dead = q0 >= n;

  TileDma<TL, D, COL_NT> dma;
  dma.init();
  dma.issue(kbuf[0], K, 0, n);
  for (int kb = 0; kb < nkb; ++kb) {
    dma_wait();
    if ((kb & 7) == 7) {
      if (__syncthreads_and(dead)) break;
    } else {
      __syncthreads();
    }
    if (kb + 1 < nkb) dma.issue(kbuf[(kb + 1) & 1], K, (kb + 1) * BLK, n);
    if (dead) continue;
    bool any = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j0 = kb * BLK + 32 * h;
      if (j0 >= n || (a.causal && j0 > last)) continue;
      f32x16 s = zero16();
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        s = M::mma(lds_row_frag_pad<E, D>(kbuf[kb & 1], 32 * h + (lane & 31), kk), qf[kk], s);
      if (j0 + 31 >= n || (a.causal && j0 + 31 > q0)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = j0 + crow(r);
          if (!(j < n && (!a.causal || j <= i))) s[r] = -INFINITY;
        }
      }
      float z[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if constexpr (PRECISE)
          z[r] = precise_relu_z<D>(row_ok, c, s[r], tau, band, tau64,
                                   reinterpret_cast<const float*>(Q) + (size_t)i * D,
                                   reinterpret_cast<const float*>(K) + (size_t)(j0 + crow(r)) * D, a.c64);
        else
          z[r] = relu_z(c, s[r], tau);
      }
#pragma unroll
      for (int r0 = 0; r0 < 16; r0 += 4) {
        if (fmaxf(max3f(z[r0], z[r0 + 1], z[r0 + 2]), z[r0 + 3]) > 0.f) {
#pragma unroll
          for (int r = r0; r < r0 + 4; ++r)
            if (z[r] > 0.f) {
              any = true;
              if (cnt < LIST_CAP) {
                lb->z[LIST_IDS * cnt + id] = z[r];
                lb->key[LIST_IDS * cnt + id] = (uint16_t)(j0 + crow(r));
              }
              ++cnt;
            }
        }
      }
    }
    if (__ballot(any) != 0ull && lane == 0) atomicOr(&bits[qbl][kb >> 5], 1u << (kb & 31));
    dead = __ballot(cnt > LIST_CAP) != 0ull;
  }
  dma_wait();  // a copy may be in flight when the loop was left
  int total = cnt > LIST_CAP ? LIST_ENTRIES + 1 : cnt;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) total += __shfl_xor(total, o);
  if (lane == 0) atomicAdd(&entries[qbl], total);
  if (lb) {
    lb->count[id] = (uint8_t)min(cnt, LIST_CAP);
    if (half == 0 && row_ok) lb->tau[row] = tau;
  }
  __syncthreads();
  if (lb && (w & 1) == 0 && lane == 0) {
    int blocks = 0;
    for (int x = 0; x < (T + 31) / 32; ++x) blocks += __popc(bits[qbl][x]);
    a.use[(size_t)bh * T + qb] = list_use(entries[qbl], blocks, T, sizeof(E) == 4);
  }
}

// ------------------------------------------------------------------ dK dV

// The number of the T query blocks of head bh that are sorted for the list
// kernel.  Every thread of the workgroup.
template <int NT>
__device__ __forceinline__ int sorted_blocks(const Buckets& b, int bh, int T) {
  if (((const ci32*)b.heads)[bh] == 0) return 0;
  const int32_t* used = b.used + (size_t)bh * T;
  int sorted = 0;
  for (int x0 = 0; x0 < T; x0 += NT) {
    const int x = x0 + (int)threadIdx.x;
    sorted += __syncthreads_count(x < T && (used[min(x, T - 1)] & SORTED) != 0);
  }
  return __builtin_amdgcn_readfirstlane(sorted);
}

// The query blocks of list[0 .. cnt) (without tables: first, first + 1, ...)
// that have no element lists, in order, in out (in LDS); returns their number.
// Every thread of the workgroup.
template <int NT>
__device__ int unlisted_blocks(const int32_t* list, int first, int cnt, const int32_t* used, uint16_t* out) {
  __shared__ int wcount[NT / 64];
  int total = 0;
  for (int e0 = 0; e0 < cnt; e0 += NT) {
    const int e = e0 + (int)threadIdx.x;
    const int qb = e < cnt ? (list ? list[e] : first + e) : 0;
    const bool b = e < cnt && !(used[qb] & SORTED);
    const unsigned long long m = __ballot(b);
    __syncthreads();  // wcount of the round before has been read
    if (lane_id() == 0) wcount[wave_id()] = __popcll(m);
    __syncthreads();
    int at = total;
#pragma unroll
    for (int x = 0; x < NT / 64; ++x) {
      if (x < wave_id()) at += wcount[x];
      total += wcount[x];
    }
    if (b) out[at + lanes_below(m)] = (uint16_t)qb;
  }
  __syncthreads();
  return total;
}

template <typename E, int D, int GK>
__global__ __launch_bounds__(BWD_NT) void dkdv_kernel(BwdArgs a) {
  using TL = Tile<E, D>;
  using M = Mma<E>;
  constexpr int KS = D / M::KW;
  constexpr int NTD = D / 32;
  constexpr int PS = perm_steps<E>();
  __shared__ __attribute__((aligned(16))) E qbuf[2][TL::ELEMS];
  __shared__ __attribute__((aligned(16))) E dobuf[2][TL::ELEMS];
  __shared__ __attribute__((aligned(16))) float tau_s[2][BLK];
  __shared__ __attribute__((aligned(16))) float del_s[2][BLK];

  const int lane = lane_id(), w = wave_id();
  const int n = a.n, T = a.T;
  const int bh = blockIdx.x % a.BH;
  const int kb = blockIdx.x / a.BH;  // causal: small kb has the longest list
  const int k0 = kb * BLK + 32 * w;
  const int j = k0 + (lane & 31);
  const bool wave_ok = k0 < n;
  const size_t head = (size_t)bh * n * D;
  const E* Qg = static_cast<const E*>(a.q) + head;
  const E* Kg = static_cast<const E*>(a.k) + head;
  const E* Vg = static_cast<const E*>(a.v) + head;
  const E* dOg = static_cast<const E*>(a.dout) + head;
  const float* taug = a.tau + (size_t)bh * n;
  const float* delg = a.delta + (size_t)bh * n;
  const float c = a.c, g = a.gamma;
  constexpr bool PRECISE = precise_path<E, GK>();

  // Without tables (the no-mask mode) every valid query block is visited.
  // With element lists only the query blocks without them are: their entries
  // are compacted into `unlisted` first, and a key block that has none is
  // left to the list kernel.
  const bool dense = a.k_index == nullptr;
  const int32_t* list = dense ? nullptr : a.k_index + ((size_t)bh * T + kb) * T;
  int cnt = dense ? (a.causal ? T - kb : T) : a.k_count[(size_t)bh * T + kb];
  __shared__ uint16_t unlisted[LIST_MAX_SEQLEN / BLK];
  const int sorted = a.lists ? sorted_blocks<BWD_NT>(a.buckets, bh, T) : 0;
  if (a.lists && sorted == T) return;
  const bool some = sorted > 0;
  if (some) {
    cnt = unlisted_blocks<BWD_NT>(list, a.causal ? kb : 0, cnt, a.buckets.used + (size_t)bh * T, unlisted);
    if (cnt == 0) return;
  }
  auto qb_of = [&](int e) { return some ? (int)unlisted[e] : dense ? (a.causal ? kb + e : e) : list[e]; };

  typename M::frag kf[KS], vf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    kf[kk] = load_row_frag_global<E, D>(Kg, j, n, kk);
    vf[kk] = load_row_frag_global<E, D>(Vg, j, n, kk);
  }

  f32x16 dk[NTD], dv[NTD];
#pragma unroll
  for (int t = 0; t < NTD; ++t) {
    dk[t] = zero16();
    dv[t] = zero16();
  }

  // One 32-query half of the staged block against this wave's 32 keys:
  // S = Q K^T, dP = dO V^T (rows = queries), then dV += P^T dO, dK += dS^T Q.
  // Masked sub-tiles set invalid scores to -inf first (the clamp of
  // [x - tau]_+ then gives exactly 0), so one code path updates dK and dV.
  auto block = [&](bool masked, const E* qt, const E* dt, const float* ts, const float* ds_,
                   int qh, int i0) {
    f32x16 s = zero16(), dp = zero16();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      s = M::mma(lds_row_frag<E, D>(qt, 32 * qh + (lane & 31), kk), kf[kk], s);
      dp = M::mma(lds_row_frag<E, D>(dt, 32 * qh + (lane & 31), kk), vf[kk], dp);
    }
    if (masked) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = i0 + crow(r);
        if (!(i < n && j < n && (!a.causal || j <= i))) s[r] = -INFINITY;
      }
    }
    float p[16], dsv[16];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      // rows 8 g4 + 4h + (0..3) of this half: one 16-byte read each for tau, delta
      const int q4 = 32 * qh + 8 * g4 + 4 * (lane >> 5);
      const f32x4 tq = *reinterpret_cast<const f32x4*>(ts + q4);
      const f32x4 dq4 = *reinterpret_cast<const f32x4*>(ds_ + q4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * g4 + e;
        float zp;
        if constexpr (PRECISE) {
          // fp64 z near the support edge (ea_common.h); invalid pairs hold -inf
          const int i = i0 + crow(r);
          const bool ok = i < n && j < n;
          const float band = PRECISE_BAND * fmaxf(1.f, fabsf(tq[e]));
          const float raw = fmaf(c, s[r], -tq[e]);
          double t64 = tq[e];
          if (ok && fabsf(raw) < band && a.tau_lo) t64 += (double)a.tau_lo[(size_t)bh * n + i];
          zp = precise_relu_z<D>(ok, c, s[r], tq[e], band, t64,
                                 reinterpret_cast<const float*>(Qg) + (size_t)i * D,
                                 reinterpret_cast<const float*>(Kg) + (size_t)j * D, a.c64);
        } else {
          zp = relu_z(c, s[r], tq[e]);
        }
        float u;
        Gamma<GK>::pu(zp, g, p[r], u);
        dsv[r] = u * (dp[r] - dq4[e]);
      }
    }
#pragma unroll
    for (int t = 0; t < PS; ++t) {
      const typename M::frag pa = M::pack(p, t);
      typename M::frag dh, dl;
      M::pack_split(dsv, t, dh, dl);
#pragma unroll
      for (int nt = 0; nt < NTD; ++nt) {
        dv[nt] = M::mma(pa, lds_perm_frag<E, D>(dt, 32 * nt, 32 * qh, t), dv[nt]);
        const typename M::frag qb_ = lds_perm_frag<E, D>(qt, 32 * nt, 32 * qh, t);
        dk[nt] = M::mma(dh, qb_, dk[nt]);
        if constexpr (!M::exact_operands) dk[nt] = M::mma(dl, qb_, dk[nt]);
      }
    }
  };

  float tv = 0.f, dlv = 0.f;
  DmaPlan<E, D, BWD_NT> dma;
  dma.init();
  auto issue = [&](int e) {
    const int qb = qb_of(e);
    dma.issue(qbuf[e & 1], Qg, qb * BLK, n);
    dma.issue(dobuf[e & 1], dOg, qb * BLK, n);
    if (threadIdx.x < BLK) {
      const int r = min(qb * BLK + (int)threadIdx.x, n - 1);
      tv = taug[r];
      dlv = delg[r];
    }
  };
  if (cnt > 0) issue(0);
  for (int e = 0; e < cnt; ++e) {
    dma_wait();
    if (threadIdx.x < BLK) {
      tau_s[e & 1][threadIdx.x] = tv;
      del_s[e & 1][threadIdx.x] = dlv;
    }
    __syncthreads();
    const int qb = qb_of(e);
    if (e + 1 < cnt) issue(e + 1);
    if (!wave_ok) continue;
    const E* qt = qbuf[e & 1];
    const E* dt = dobuf[e & 1];
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) {
      const int i0 = qb * BLK + 32 * qh;
      if (i0 >= n || (a.causal && k0 > i0 + 31)) continue;
      const bool masked = i0 + 31 >= n || k0 + 31 >= n || (a.causal && k0 + 31 > i0);
      block(masked, qt, dt, tau_s[e & 1], del_s[e & 1], qh, i0);
    }
  }

  if (!wave_ok) return;
  float* dK = a.dk + head;
  float* dV = a.dv + head;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int key = k0 + crow(r);
    if (key < n) {
#pragma unroll
      for (int nt = 0; nt < NTD; ++nt) {
        const size_t off = (size_t)key * D + 32 * nt + (lane & 31);
        dK[off] = a.scale * dk[nt][r];
        dV[off] = dv[nt][r];
      }
    }
  }
}

// ------------------------------------------------------- dK dV, bf16 inputs

// Eight waves over two adjacent key blocks (2m and 2m + 1).  Wave w owns key
// block 2m + (w >> 2), key half kh = (w >> 1) & 1 (32 keys, as above) and
// column half ch = w & 1 of dK and dV.  For each staged query block the wave
// forms S and dP of its keys against query half ch only, turns them into the
// operands P, dS_hi and dS_lo of the permuted contractions and posts those
// through LDS; its partner (same keys, other column half) posts the other
// query half.  Each wave then accumulates dV and dK for its columns over
// both query halves.  Half the accumulators and no repeated products let
// two waves share each SIMD, while every product is formed once.  The two
// key blocks visit the union of their query-block lists (both ascending);
// the waves of a key block that does not list the staged query block only
// keep the barriers.
//
// The Q and dO tiles (with their tau and delta) go through three LDS stages,
// so each copy has two steps to land, and the barriers wait only for LDS
// traffic: a plain workgroup barrier would also wait for the copies in
// flight.  The tables are read by scalar loads for the same reason.
constexpr int BWD2_NT = 512;

template <int D, int GK>
__global__ __launch_bounds__(BWD2_NT, 2) void dkdv2_kernel(BwdArgs a) {
  using E = __bf16;
  using TL = Tile<E, D>;
  using M = Mma<E>;
  using F = typename M::frag;
  constexpr int KS = D / M::KW;
  constexpr int NTH = D / 64;  // 32-column output tiles per wave
  constexpr int PS = perm_steps<E>();
  // three stages: block e is read while e + 1 and e + 2 are in flight
  __shared__ __attribute__((aligned(16))) E qbuf[3][TL::ELEMS];
  __shared__ __attribute__((aligned(16))) E dobuf[3][TL::ELEMS];
  __shared__ __attribute__((aligned(16))) float tau_s[3][BLK];
  __shared__ __attribute__((aligned(16))) float del_s[3][BLK];
  // operands posted by each wave: [wave][P, dS hi, dS lo][step][lane]
  __shared__ __attribute__((aligned(16))) u32x4 post[BWD2_NT / 64][3][PS][64];

  const int lane = lane_id(), w = wave_id();
  const int kh = (w >> 1) & 1, ch = w & 1;
  const int n = a.n, T = a.T;
  const int bh = blockIdx.x % a.BH;
  const int kbA = 2 * (blockIdx.x / a.BH);  // causal: small key blocks have the longest lists
  const int kbB = kbA + 1;
  const bool mineA = (w >> 2) == 0;
  const int k0 = (mineA ? kbA : kbB) * BLK + 32 * kh;
  const int j = k0 + (lane & 31);
  const bool wave_ok = k0 < n;
  const size_t head = (size_t)bh * n * D;
  const E* Qg = static_cast<const E*>(a.q) + head;
  const E* Kg = static_cast<const E*>(a.k) + head;
  const E* Vg = static_cast<const E*>(a.v) + head;
  const E* dOg = static_cast<const E*>(a.dout) + head;
  [[maybe_unused]] const float* taug = a.tau + (size_t)bh * n;  // read by tile copies
  [[maybe_unused]] const float* delg = a.delta + (size_t)bh * n;
  const float c = a.c, g = a.gamma;

  // Query-block lists of the two key blocks (without tables, in the no-mask
  // mode, every valid query block), merged in ascending order.
  const bool dense = a.k_index == nullptr;
  const ci32* kcount = (const ci32*)a.k_count;
  const ci32* kindex = (const ci32*)a.k_index;
  __shared__ uint16_t unlisted[2][LIST_MAX_SEQLEN / BLK];
  const int sorted = a.lists ? sorted_blocks<BWD2_NT>(a.buckets, bh, T) : 0;
  if (a.lists && sorted == T) return;
  const bool some = sorted > 0;
  auto count_of = [&](int kb) {
    if (kb >= T) return 0;
    return dense ? (a.causal ? T - kb : T) : kcount[(size_t)bh * T + kb];
  };
  auto entry_of = [&](auto left, int kb, int e) {
    if constexpr (decltype(left)::value) return __builtin_amdgcn_readfirstlane((int)unlisted[kb - kbA][e]);
    return dense ? (a.causal ? kb + e : e) : kindex[((size_t)bh * T + kb) * T + e];
  };
  int nA = count_of(kbA), nB = count_of(kbB);
  int pA = 0, pB = 0;
  // With element lists, only the query blocks without them (see dkdv_kernel).
  if (some) {
    const int32_t* used = a.buckets.used + (size_t)bh * T;
    const int32_t* lA = dense ? nullptr : a.k_index + ((size_t)bh * T + kbA) * T;
    const int32_t* lB = dense ? nullptr : a.k_index + ((size_t)bh * T + min(kbB, T - 1)) * T;
    nA = unlisted_blocks<BWD2_NT>(lA, a.causal ? kbA : 0, nA, used, unlisted[0]);
    nB = unlisted_blocks<BWD2_NT>(lB, a.causal ? kbB : 0, nB, used, unlisted[1]);
    if (nA == 0 && nB == 0) return;
    // (scalar registers: they steer the loop below)
    nA = __builtin_amdgcn_readfirstlane(nA);
    nB = __builtin_amdgcn_readfirstlane(nB);
  }
  // the next query block of the union, and whether each key block lists it
  auto next = [&](auto left, int& qb, bool& inA, bool& inB) {
    const int hA = pA < nA ? entry_of(left, kbA, pA) : T;
    const int hB = pB < nB ? entry_of(left, kbB, pB) : T;
    qb = min(hA, hB);
    inA = hA == qb;
    inB = hB == qb;
    pA += inA ? 1 : 0;
    pB += inB ? 1 : 0;
    return qb < T;
  };

  F kf[KS], vf[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    kf[kk] = load_row_frag_global<E, D>(Kg, j, n, kk);
    vf[kk] = load_row_frag_global<E, D>(Vg, j, n, kk);
  }

  f32x16 dk[NTH], dv[NTH];
#pragma unroll
  for (int t = 0; t < NTH; ++t) {
    dk[t] = zero16();
    dv[t] = zero16();
  }

  // S = Q K^T, dP = dO V^T of query half qh (rows = queries) for this wave's
  // keys; masked sub-tiles set invalid scores to -inf (then P = dS = 0).
  auto operands = [&](const E* qt, const E* dt, const float* ts, const float* ds_, int qh,
                      bool masked, int i0, F* pa, F* dh, F* dl) {
    f32x16 s = zero16(), dp = zero16();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      s = M::mma(lds_row_frag<E, D>(qt, 32 * qh + (lane & 31), kk), kf[kk], s);
      dp = M::mma(lds_row_frag<E, D>(dt, 32 * qh + (lane & 31), kk), vf[kk], dp);
    }
    if (masked) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = i0 + crow(r);
        if (!(i < n && j < n && (!a.causal || j <= i))) s[r] = -INFINITY;
      }
    }
    float p[16], dsv[16];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int q4 = 32 * qh + 8 * g4 + 4 * (lane >> 5);
      const f32x4 tq = *reinterpret_cast<const f32x4*>(ts + q4);
      const f32x4 dq4 = *reinterpret_cast<const f32x4*>(ds_ + q4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * g4 + e;
        const float zp = relu_z(c, s[r], tq[e]);
        float u;
        Gamma<GK>::pu(zp, g, p[r], u);
        dsv[r] = u * (dp[r] - dq4[e]);
      }
    }
#pragma unroll
    for (int t = 0; t < PS; ++t) {
      pa[t] = M::pack(p, t);
      M::pack_split(dsv, t, dh[t], dl[t]);
    }
  };
  // dV += P^T dO and dK += dS^T Q over query half qh, this wave's columns
  auto accum = [&](const E* qt, const E* dt, int qh, const F* pa, const F* dh, const F* dl) {
#pragma unroll
    for (int t = 0; t < PS; ++t) {
#pragma unroll
      for (int nt = 0; nt < NTH; ++nt) {
        const int col0 = 32 * (ch * NTH + nt);
        dv[nt] = M::mma(pa[t], lds_perm_frag<E, D>(dt, col0, 32 * qh, t), dv[nt]);
        const F qb_ = lds_perm_frag<E, D>(qt, col0, 32 * qh, t);
        dk[nt] = M::mma(dh[t], qb_, dk[nt]);
        dk[nt] = M::mma(dl[t], qb_, dk[nt]);
      }
    }
  };
  auto half_valid = [&](int i0) { return !(i0 >= n || (a.causal && k0 > i0 + 31)); };
  auto half_masked = [&](int i0) {
    return i0 + 31 >= n || k0 + 31 >= n || (a.causal && k0 + 31 > i0);
  };

  using Plan = DmaPlan<E, D, BWD2_NT>;
  static_assert(Plan::NI % Plan::NW == 0 && 2 * Plan::PER + 2 <= 15, "copy counts");
  Plan dma;
  dma.init();
  // Copies of query block qb into stage b: the Q and dO tiles, and (wave 0)
  // its tau and delta values, all by global_load_lds.
  auto issue = [&](int qb, int b) {
    dma.issue(qbuf[b], Qg, qb * BLK, n);
    dma.issue(dobuf[b], dOg, qb * BLK, n);
#if defined(__HIP_DEVICE_COMPILE__)
    if (w == 0) {
      const int r = min(qb * BLK + lane, n - 1);
      __builtin_amdgcn_global_load_lds(taug + r, to_lds(&tau_s[b][0]), 4, 0, 0);
      __builtin_amdgcn_global_load_lds(delg + r, to_lds(&del_s[b][0]), 4, 0, 0);
    }
#endif
  };
  // Workgroup barrier for LDS traffic only: this wave's LDS operations
  // complete first, but copies still in flight are not waited for (the
  // plain barrier would also wait for every global load, so the next
  // stages' copies would have to land first).
  auto lds_barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  // Waits until every copy but those of the latest issue has landed (the
  // counter completes in issue order; wave 0 issues two more per stage).
  auto wait_all_but_latest = [&]() {
    if (w == 0) {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * Plan::PER + 2));
    } else {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (2 * Plan::PER));
    }
  };
  // S, dP, P, dS of query half ch (kept for this wave, posted for its partner)
  F pa[PS], dh[PS], dl[PS];
  auto phase1 = [&](int qb, int b, int tb) {
    const int i0 = qb * BLK + 32 * ch;
    if (!half_valid(i0)) return;
    operands(qbuf[b], dobuf[b], tau_s[tb], del_s[tb], ch, half_masked(i0), i0, pa, dh, dl);
#pragma unroll
    for (int t = 0; t < PS; ++t) {
      post[w][0][t][lane] = __builtin_bit_cast(u32x4, pa[t]);
      post[w][1][t][lane] = __builtin_bit_cast(u32x4, dh[t]);
      post[w][2][t][lane] = __builtin_bit_cast(u32x4, dl[t]);
    }
  };
  // both query halves into this wave's columns: the partner's half first
  auto phase2 = [&](int qb, int b) {
    if (half_valid(qb * BLK + 32 * (ch ^ 1))) {
      F xa[PS], xh[PS], xl[PS];
#pragma unroll
      for (int t = 0; t < PS; ++t) {
        xa[t] = __builtin_bit_cast(F, post[w ^ 1][0][t][lane]);
        xh[t] = __builtin_bit_cast(F, post[w ^ 1][1][t][lane]);
        xl[t] = __builtin_bit_cast(F, post[w ^ 1][2][t][lane]);
      }
      accum(qbuf[b], dobuf[b], ch ^ 1, xa, xh, xl);
    }
    if (half_valid(qb * BLK + 32 * ch)) accum(qbuf[b], dobuf[b], ch, pa, dh, dl);
  };

  // `left`: only the query blocks left in `unlisted`, a loop of its own, so
  // that the one over whole tables keeps its scalar loads alone.
  auto run = [&](auto left) {
    // Union entries e (stage b0), e + 1 and e + 2 (in flight).
    int q0 = 0, q1 = 0;
    bool a0 = false, b0_ = false, a1 = false, b1_ = false;
    bool h0 = next(left, q0, a0, b0_);
    bool h1 = h0 && next(left, q1, a1, b1_);
    if (h0) issue(q0, 0);
    if (h1) issue(q1, 1);
    int st = 0;
    while (h0) {
      int q2 = 0;
      bool a2 = false, b2_ = false;
      const bool h2 = h1 && next(left, q2, a2, b2_);
      if (h1) {
        wait_all_but_latest();
      } else {
        dma_wait();
      }
      // block q0 is staged (each wave waited for its own copies); every wave
      // is done with the previous step, whose stage receives block q2
      lds_barrier();
      if (h2) issue(q2, st == 0 ? 2 : st - 1);
      const bool act = wave_ok && (mineA ? a0 : b0_);
      if (act) phase1(q0, st, st);
      lds_barrier();  // the posted operands are visible
      if (act) phase2(q0, st);
      q0 = q1;
      a0 = a1;
      b0_ = b1_;
      h0 = h1;
      q1 = q2;
      a1 = a2;
      b1_ = b2_;
      h1 = h2;
      st = st == 2 ? 0 : st + 1;
    }
  };
  if (some)
    run(std::true_type{});
  else
    run(std::false_type{});

  if (!wave_ok) return;
  float* dK = a.dk + head;
  float* dV = a.dv + head;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int key = k0 + crow(r);
    if (key < n) {
#pragma unroll
      for (int nt = 0; nt < NTH; ++nt) {
        const size_t off = (size_t)key * D + 32 * (ch * NTH + nt) + (lane & 31);
        dK[off] = a.scale * dk[nt][r];
        dV[off] = dv[nt][r];
      }
    }
  }
}

// ----------------------------------------------- dK dV, listed query blocks

// dK and dV of one key block from the entries of its listed query blocks.
// The entries of up to LK_NT query blocks at a time are copied into LDS (at
// most LK_CHUNK per round), sorted by key (counting sort, deterministic as in
// prep_kernel), and dealt out in equal, consecutive shares to the groups of
// lanes, whatever their keys: a key that many queries attend to is shared by
// several groups.  A group adds up dV and dK of one key after another in
// registers (p dO_i and dS Q_i, with dP = <dO_i, V_j> summed over its lanes).
// The group in whose share a key starts owns it: groups whose share starts
// inside a key post their part of it in LDS, and the owner adds the parts in
// order.  Per entry this reads one row of dO and one of Q from L2.
constexpr int LK_NT = 256;
constexpr int LK_CHUNK = 2048;

template <typename E, int D, int GK>
__global__ __launch_bounds__(LK_NT, 2) void dkdv_lists_kernel(BwdArgs a) {
  using R = RowGroup<E, D>;
  constexpr int VPL = R::VPL, LPR = R::LPR, NG = LK_NT / LPR, W = LK_NT / 64;
  __shared__ uint32_t code[LK_CHUNK];   // (query row << 6) | key
  __shared__ float zv[LK_CHUNK];
  __shared__ uint16_t order[LK_CHUNK];
  __shared__ int cursor[W][BLK];
  __shared__ int kstart[BLK + 1];
  __shared__ int wsum[W];
  __shared__ uint16_t run_qb[LK_NT], run_from[LK_NT], run_num[LK_NT];
  __shared__ int run_at[LK_NT];
  __shared__ __attribute__((aligned(16))) u32x4 vt[BLK * LPR];        // rows of V
  __shared__ __attribute__((aligned(16))) float part[NG][2 * D];      // dV, dK of a share's leading key
  const int t = threadIdx.x, lane = lane_id(), w = wave_id(), sub = lane % LPR, grp = t / LPR;
  const int n = a.n, T = a.T;
  int bh, kb;
  head_major(blockIdx.x, a.BH, T, bh, kb);
  const size_t head = (size_t)bh * n * D;
  const E* Q = static_cast<const E*>(a.q) + head;
  const E* V = static_cast<const E*>(a.v) + head;
  const E* dO = static_cast<const E*>(a.dout) + head;
  const float* del = a.delta + (size_t)bh * n;
  const int k0 = kb * BLK;
  const bool dense = a.k_index == nullptr;  // no tables: every valid query block
  const int32_t* list = dense ? nullptr : a.k_index + ((size_t)bh * T + kb) * T;
  const int cnt = dense ? (a.causal ? T - kb : T) : a.k_count[(size_t)bh * T + kb];
  auto qb_of = [&](int e) { return dense ? (a.causal ? kb + e : e) : list[e]; };
  const int32_t* used = a.buckets.used + (size_t)bh * T;

  const int sorted = sorted_blocks<LK_NT>(a.buckets, bh, T);
  if (sorted == 0) return;
  // whether the other dK/dV kernel wrote this key block (some query block of
  // its list is not sorted): the first round then adds to it as the later
  // ones do
  bool add = false;
  if (sorted < T) {
    bool other = false;
    for (int e = t; e < cnt; e += LK_NT) other |= !(used[qb_of(e)] & SORTED);
    add = __syncthreads_or(other);
  }
#pragma unroll
  for (int r = grp; r < BLK; r += NG) vt[r * LPR + sub] = R::load(V, (uint32_t)min(k0 + r, n - 1));

  // dK and dV of key kl, this lane's columns
  auto put = [&](int kl, const float (&dv)[VPL], const float (&dk)[VPL]) {
    if (k0 + kl >= n) return;
    const size_t at = head + (size_t)(k0 + kl) * D + sub * VPL;
#pragma unroll
    for (int d = 0; d < VPL; d += 4) {
      f32x4 x = {dv[d], dv[d + 1], dv[d + 2], dv[d + 3]};
      f32x4 y = {a.scale * dk[d], a.scale * dk[d + 1], a.scale * dk[d + 2], a.scale * dk[d + 3]};
      if (add) {
        x += *reinterpret_cast<const f32x4*>(a.dv + at + d);
        y += *reinterpret_cast<const f32x4*>(a.dk + at + d);
      }
      *reinterpret_cast<f32x4*>(a.dv + at + d) = x;
      *reinterpret_cast<f32x4*>(a.dk + at + d) = y;
    }
  };

  int e0 = 0;
  do {
    // The runs of this batch: query block, place in its buckets, length, and
    // (run_at) the sum of the lengths before it.
    const int e = e0 + t;
    int qb = 0, from = 0, num = 0;
    if (e < cnt) {
      qb = qb_of(e);
      if (used[qb] & SORTED) {
        const uint16_t* off = a.buckets.off + ((size_t)bh * T + qb) * (size_t)(T + 1) + kb;
        from = off[0];
        num = off[1] - from;
      }
    }
    int incl = num;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    __syncthreads();  // wsum and the runs of the batch before have been read
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int at = incl - num, total = 0;
#pragma unroll
    for (int x = 0; x < W; ++x) {
      if (x < w) at += wsum[x];
      total += wsum[x];
    }
    run_qb[t] = (uint16_t)qb;
    run_from[t] = (uint16_t)from;
    run_num[t] = (uint16_t)num;
    run_at[t] = at;
    __syncthreads();
    // tp threads (a power of two) copy one run
    const int runs = max(min(cnt - e0, LK_NT), 1);
    int tp = 1;
    while (2 * tp * runs <= LK_NT) tp *= 2;
    const int run = t / tp;
    int c0 = 0;  // entries [c0, c0 + LK_CHUNK) of the batch in this round
    do {
      const int M = min(total - c0, LK_CHUNK);
      if (run < runs) {
        const int rq = run_qb[run], ra = run_at[run], rn = min((int)run_num[run], c0 + LK_CHUNK - ra);
        const size_t src = ((size_t)bh * T + rq) * LIST_ENTRIES + run_from[run];
        constexpr int B = 4;
        for (int x0 = max(0, c0 - ra) + t % tp; x0 < rn; x0 += B * tp) {
          int cd[B];
          float z[B];
#pragma unroll
          for (int u = 0; u < B; ++u) {
            const int x = min(x0 + u * tp, rn - 1);
            cd[u] = a.buckets.code[src + x];
            z[u] = a.buckets.z[src + x];
          }
#pragma unroll
          for (int u = 0; u < B; ++u) {
            const int x = x0 + u * tp;
            if (x < rn) {
              code[ra + x - c0] = ((uint32_t)(rq * BLK + (cd[u] >> 6)) << 6) | (uint32_t)(cd[u] & 63);
              zv[ra + x - c0] = z[u];
            }
          }
        }
      }
      (&cursor[0][0])[t] = 0;  // W * BLK = LK_NT counters
      __syncthreads();
      // sort by key: wave w takes entries [w * q, (w + 1) * q)
      const int q = (M + W - 1) / W, b0 = w * q, b1 = min(M, b0 + q);
      for (int x = b0 + lane; x < b1; x += 64) atomicAdd(&cursor[w][code[x] & 63], 1);
      __syncthreads();
      if (w == 0) {
        int s = 0;
#pragma unroll
        for (int x = 0; x < W; ++x) s += cursor[x][lane];
        int in = s;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int v = __shfl_up(in, o);
          if (lane >= o) in += v;
        }
        int p = in - s;
        kstart[lane] = p;
        if (lane == 63) kstart[BLK] = in;
#pragma unroll
        for (int x = 0; x < W; ++x) {
          const int v = cursor[x][lane];
          cursor[x][lane] = p;
          p += v;
        }
      }
      __syncthreads();
      for (int x = b0; x < b1; x += 64) {
        const bool ok = x + lane < b1;
        const int key = ok ? (int)(code[x + lane] & 63u) : 0;
        const unsigned long long m = same_key(key, 6, __ballot(ok));
        if (ok) {
          const int rank = lanes_below(m);
          const int p = cursor[w][key] + rank;
          if (rank == __popcll(m) - 1) cursor[w][key] = p + 1;
          order[p] = (uint16_t)(x + lane);
        }
      }
      __syncthreads();

      // this group's share of the sorted entries
      const int share = (M + NG - 1) / NG;
      const int s0 = grp * share, s1 = min(M, s0 + share);
      float dv[VPL] = {}, dk[VPL] = {};
      int cur = -1;          // the key being added up
      bool lead = false;     // it started in an earlier share
      bool owe = false;      // after the loop: `cur` is this group's, unfinished
      auto post_part = [&]() {
#pragma unroll
        for (int d = 0; d < VPL; ++d) {
          part[grp][sub * VPL + d] = dv[d];
          part[grp][D + sub * VPL + d] = dk[d];
        }
      };
      // batches of U entries, the next one's rows in flight meanwhile (past
      // the end of the share its last entry again)
      constexpr int U = 4;
      u32x4 ow[U], qw[U];
      uint32_t cd[U];
      float z[U], dl[U];
      auto fetch = [&](int p0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int o = (int)order[max(min(p0 + u, s1 - 1), 0)];
          cd[u] = code[o];
          z[u] = zv[o];
          ow[u] = R::load(dO, cd[u] >> 6);
          qw[u] = R::load(Q, cd[u] >> 6);
          dl[u] = del[cd[u] >> 6];
        }
      };
      if (M > 0) fetch(s0);
      for (int p0 = s0; __ballot(p0 < s1) != 0ull; p0 += U) {
        u32x4 ow0[U], qw0[U];
        uint32_t cd0[U];
        float z0[U], dl0[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ow0[u] = ow[u];
          qw0[u] = qw[u];
          cd0[u] = cd[u];
          z0[u] = z[u];
          dl0[u] = dl[u];
        }
        fetch(p0 + U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (p0 + u < s1) {
            const int kl = (int)(cd0[u] & 63u);
            if (kl != cur) {
              if (cur >= 0) {
                if (lead)
                  post_part();
                else
                  put(cur, dv, dk);
              }
              cur = kl;
              lead = kstart[kl] < s0;
#pragma unroll
              for (int d = 0; d < VPL; ++d) dv[d] = dk[d] = 0.f;
            }
            float x[VPL], y[VPL];
            R::unpack(ow0[u], x);
            R::unpack(vt[kl * LPR + sub], y);
            float dp = 0.f, pp, uu;
#pragma unroll
            for (int d = 0; d < VPL; ++d) dp = fmaf(x[d], y[d], dp);
            dp = R::sum(dp);
            Gamma<GK>::pu(z0[u], a.gamma, pp, uu);
            const float ds = uu * (dp - dl0[u]);
            R::unpack(qw0[u], y);
#pragma unroll
            for (int d = 0; d < VPL; ++d) {
              dv[d] = fmaf(pp, x[d], dv[d]);
              dk[d] = fmaf(ds, y[d], dk[d]);
            }
          }
        }
      }
      if (cur >= 0) {
        if (lead)
          post_part();
        else if (kstart[cur + 1] <= s1)
          put(cur, dv, dk);
        else
          owe = true;
      }
      __syncthreads();
      if (owe) {
        for (int g = grp + 1; g * share < kstart[cur + 1]; ++g) {
#pragma unroll
          for (int d = 0; d < VPL; ++d) {
            dv[d] += part[g][sub * VPL + d];
            dk[d] += part[g][D + sub * VPL + d];
          }
        }
        put(cur, dv, dk);
      }
      if (!add) {  // keys without entries
        const float zero[VPL] = {};
        for (int kl = grp; kl < BLK; kl += NG)
          if (kstart[kl] == kstart[kl + 1]) put(kl, zero, zero);
      }
      add = true;
      __syncthreads();
      c0 += LK_CHUNK;
    } while (c0 < total);
    e0 += LK_NT;
  } while (e0 < cnt);
}

// --------------------------------------------------------------------- dQ

constexpr int DQ_NT = 256;

// One 64-row query block per workgroup of 4 waves: wave w takes query half
// qh = w % 2 and, of every listed key block, key half kh = w / 2, so each
// wave holds only its 32 query rows and one partial dQ; the two key-half
// partials are summed through LDS at the end.  Halving the per-wave state
// lets two waves share each SIMD.  At d = 128 a wave raises its issue
// priority over its dQ products, so that the two waves of a SIMD drift
// apart (B1 H16 n8192: 0.905 against 0.922 ms at alpha = 1.5, c = 1, 0.505
// against 0.531 at c = 16, 0.925 against 0.941 at alpha = 1.25, c = 1, 0.806
// against 0.844 at alpha = 2, c = 1); at d = 64 that was slower (0.256
// against 0.252 ms on B1 H8 n16384 causal).
// dQ of a query block from its element lists (see gather_fwd): dP = <dO_i,
// V_j> summed over a group's lanes, then dQ_i += dS K_j in registers.  Per
// entry this reads one row of V and one of K from L2.
template <typename E, int D, int GK>
__device__ __forceinline__ void gather_dq(const BwdArgs& a, const ListBlock& lb, int bh, int qb) {
  using R = RowGroup<E, D>;
  constexpr int VPL = R::VPL, LPR = R::LPR, BATCH = 8;
  const int lane = lane_id(), w = wave_id(), sub = lane % LPR;
  const int n = a.n;
  const size_t head = (size_t)bh * n * D;
  const E* K = static_cast<const E*>(a.k) + head;
  const E* V = static_cast<const E*>(a.v) + head;
  const E* dO = static_cast<const E*>(a.dout) + head;
  for (int r0 = w * R::GROUPS; r0 < BLK; r0 += 4 * R::GROUPS) {
    const int row = r0 + lane / LPR, i = qb * BLK + row;
    const int c0 = lb.count[row], cnt = c0 + lb.count[64 + row];
    const uint32_t ir = (uint32_t)min(i, n - 1);
    const float del = a.delta[(size_t)bh * n + ir];
    float go[VPL], acc[VPL] = {};
    R::unpack(R::load(dO, ir), go);
    for (int base = 0; __ballot(base < cnt) != 0ull; base += LPR) {
      float z = 0.f;
      int key = 0;
      if (cnt > 0) {
        const int e = min(base + sub, cnt - 1);
        const int at = e < c0 ? LIST_IDS * e + row : LIST_IDS * (e - c0) + 64 + row;
        key = lb.key[at];
        if (base + sub < cnt) z = lb.z[at];
      }
#pragma unroll
      for (int u0 = 0; u0 < LPR; u0 += BATCH) {
        if (u0 > 0 && __ballot(base + u0 < cnt) == 0ull) break;
        u32x4 vw[BATCH], kw[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const uint32_t j = (uint32_t)R::from(key, u0 + u);
          vw[u] = R::load(V, j);
          kw[u] = R::load(K, j);
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          float x[VPL], dp = 0.f, p, ue;
          R::unpack(vw[u], x);
#pragma unroll
          for (int d = 0; d < VPL; ++d) dp = fmaf(go[d], x[d], dp);
          dp = R::sum(dp);
          Gamma<GK>::pu(R::from(z, u0 + u), a.gamma, p, ue);
          // (nothing from the repeated entries past the end, whatever dP is)
          const float ds = ue > 0.f ? ue * (dp - del) : 0.f;
          R::unpack(kw[u], x);
#pragma unroll
          for (int d = 0; d < VPL; ++d) acc[d] = fmaf(ds, x[d], acc[d]);
        }
      }
    }
    if (i >= n) continue;
    float* dQ = a.dq + head + (size_t)i * D + sub * VPL;
#pragma unroll
    for (int d = 0; d < VPL; d += 4) {
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = cnt > 0 ? a.scale * acc[d + e] : 0.f;
      *reinterpret_cast<f32x4*>(dQ + d) = o;
    }
  }
}

template <typename E, int D, int GK>
__global__ __launch_bounds__(DQ_NT, 2) void dq_kernel(BwdArgs a) {
  using TL = Tile<E, D>;
  using M = Mma<E>;
  constexpr int KS = D / M::KW;
  constexpr int NTD = D / 32;
  constexpr int PS = perm_steps<E>();
  __shared__ __attribute__((aligned(16))) E kbuf[2][TL::ELEMS];
  __shared__ __attribute__((aligned(16))) E vbuf[2][TL::ELEMS];
  static_assert(2 * NTD * 16 * 64 * sizeof(float) <= sizeof(kbuf), "dQ exchange must fit kbuf");

  const int lane = lane_id(), w = wave_id();
  const int qh = w & 1, kh = w >> 1;
  const int n = a.n, T = a.T;
  int bh = blockIdx.x % a.BH;
  int qb = blockIdx.x / a.BH;
  if (a.lists) head_major(blockIdx.x, a.BH, T, bh, qb, head_group<E, D>(n, 2));
  if (a.causal) qb = T - 1 - qb;  // longest lists first
  if (a.lists && (a.buckets.used[(size_t)bh * T + qb] & LISTED)) {
    gather_dq<E, D, GK>(a, a.lists[(size_t)bh * T + qb], bh, qb);
    return;
  }
  const int q0 = qb * BLK + 32 * qh;
  const int i = q0 + (lane & 31);
  const bool wave_ok = q0 < n;
  const int wave_last = min(n - 1, q0 + 31);
  const size_t head = (size_t)bh * n * D;
  const E* Qg = static_cast<const E*>(a.q) + head;
  const E* Kg = static_cast<const E*>(a.k) + head;
  const E* Vg = static_cast<const E*>(a.v) + head;
  const E* dOg = static_cast<const E*>(a.dout) + head;
  const float tau = i < n ? a.tau[(size_t)bh * n + i] : 0.f;
  const float del = i < n ? a.delta[(size_t)bh * n + i] : 0.f;
  const float c = a.c, g = a.gamma;
  constexpr bool PRECISE = precise_path<E, GK>();
  // fp32 inputs, general alpha: fp64 z near the support edge (ea_common.h)
  [[maybe_unused]] const double tau64 =
      (double)tau + (PRECISE && a.tau_lo && i < n ? (double)a.tau_lo[(size_t)bh * n + i] : 0.0);
  [[maybe_unused]] const float band = PRECISE_BAND * fmaxf(1.f, fabsf(tau));

  typename M::frag qf[KS], df[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    qf[kk] = load_row_frag_global<E, D>(Qg, i, n, kk);
    df[kk] = load_row_frag_global<E, D>(dOg, i, n, kk);
  }

  // Without tables (the no-mask mode) every valid key block is visited.
  const bool dense = a.q_index == nullptr;
  const ci32* list = (const ci32*)(dense ? nullptr : a.q_index + ((size_t)bh * T + qb) * T);
  const int cnt = dense ? (a.causal ? qb + 1 : T) : ((const ci32*)a.q_count)[(size_t)bh * T + qb];
  auto kb_of = [&](int e) { return dense ? e : list[e]; };

  f32x16 dq[NTD];
#pragma unroll
  for (int t = 0; t < NTD; ++t) dq[t] = zero16();

  // 0 = no valid key for this wave, 1 = all valid, 2 = per-element masking
  auto sub_kind = [&](int j0) {
    if (!wave_ok || j0 >= n || (a.causal && j0 > wave_last)) return 0;
    if (j0 + 31 >= n || (a.causal && j0 + 31 > q0)) return 2;
    return 1;
  };

  DmaPlan<E, D, DQ_NT> dma;
  dma.init();
  auto issue = [&](int kb, int e) {
    dma.issue(kbuf[e & 1], Kg, kb * BLK, n);
    dma.issue(vbuf[e & 1], Vg, kb * BLK, n);
  };
  // key block of this step, and of the next, read a step ahead
  int kb = cnt > 0 ? kb_of(0) : 0, kb_next = cnt > 1 ? kb_of(1) : 0;
  if (cnt > 0) issue(kb, 0);
  for (int e = 0; e < cnt; ++e) {
    const int j0 = kb * BLK + 32 * kh;
    kb = kb_next;
    dma_wait();
    __syncthreads();
    if (e + 1 < cnt) issue(kb, e + 1);
    if (e + 2 < cnt) kb_next = kb_of(e + 2);
    const E* kt = kbuf[e & 1];
    const E* vt = vbuf[e & 1];
    const int kind = sub_kind(j0);
    if (kind == 0) continue;
    // S^T = K Q^T and dP^T = V dO^T for this wave's 32 keys x 32 queries
    f32x16 s = zero16(), dp = zero16();
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      s = M::mma(lds_row_frag<E, D>(kt, 32 * kh + (lane & 31), kk), qf[kk], s);
      dp = M::mma(lds_row_frag<E, D>(vt, 32 * kh + (lane & 31), kk), df[kk], dp);
    }
    if (kind == 2) {  // invalid keys -> -inf, so [x - tau]_+ is exactly 0 there
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int jj = j0 + crow(r);
        if (!(jj < n && (!a.causal || jj <= i))) s[r] = -INFINITY;
      }
    }
    float dsv[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float zp;
      if constexpr (PRECISE) {
        zp = precise_relu_z<D>(i < n, c, s[r], tau, band, tau64,
                               reinterpret_cast<const float*>(Qg) + (size_t)i * D,
                               reinterpret_cast<const float*>(Kg) + (size_t)(j0 + crow(r)) * D, a.c64);
      } else {
        zp = relu_z(c, s[r], tau);
      }
      float p, u;
      Gamma<GK>::pu(zp, g, p, u);
      dsv[r] = u * (dp[r] - del);
    }
    if constexpr (D == 128) __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int t = 0; t < PS; ++t) {
      typename M::frag dh, dl;
      M::pack_split(dsv, t, dh, dl);
#pragma unroll
      for (int nt = 0; nt < NTD; ++nt) {
        const typename M::frag kb_ = lds_perm_frag<E, D>(kt, 32 * nt, 32 * kh, t);
        dq[nt] = M::mma(dh, kb_, dq[nt]);
        if constexpr (!M::exact_operands) dq[nt] = M::mma(dl, kb_, dq[nt]);
      }
    }
    if constexpr (D == 128) __builtin_amdgcn_s_setprio(0);
  }

  // sum the two key-half partials: kh = 1 hands its accumulators over in LDS
  __syncthreads();
  float* xch = reinterpret_cast<float*>(&kbuf[0][0]);
  if (kh == 1) {
#pragma unroll
    for (int nt = 0; nt < NTD; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) xch[((qh * NTD + nt) * 16 + r) * 64 + lane] = dq[nt][r];
  }
  __syncthreads();
  if (kh == 1 || !wave_ok) return;
  float* dQ = a.dq + head;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int ir = q0 + crow(r);
    if (ir < n) {
#pragma unroll
      for (int nt = 0; nt < NTD; ++nt)
        dQ[(size_t)ir * D + 32 * nt + (lane & 31)] =
            a.scale * (dq[nt][r] + xch[((qh * NTD + nt) * 16 + r) * 64 + lane]);
    }
  }
}

template <typename E, int D>
hipError_t launch_dkdv_d(const BwdArgs& a, hipStream_t s) {
  // d = 128 bf16 takes the column-split kernel; at d = 64 (and for fp32)
  // the one-block kernel already runs two waves per SIMD without the union
  // of two query-block lists, and is faster on sparse masks.
  if constexpr (sizeof(E) == 2 && D == 128) {
    dim3 grid((unsigned)(a.BH * ((a.T + 1) / 2))), block(BWD2_NT);
    auto kernel = dkdv2_kernel<D, 0>;
    if (a.gk == 1) kernel = dkdv2_kernel<D, 1>;
    if (a.gk == 2) kernel = dkdv2_kernel<D, 2>;
    if (a.gk == 4) kernel = dkdv2_kernel<D, 4>;
    return launch_kernel(kernel, grid, block, s, a);
  }
  dim3 grid((unsigned)(a.BH * a.T)), block(BWD_NT);
  auto kernel = dkdv_kernel<E, D, 0>;
  if (a.gk == 1) kernel = dkdv_kernel<E, D, 1>;
  if (a.gk == 2) kernel = dkdv_kernel<E, D, 2>;
  if (a.gk == 4) kernel = dkdv_kernel<E, D, 4>;
  return launch_kernel(kernel, grid, block, s, a);
}

template <typename E, int D>
hipError_t launch_dq_d(const BwdArgs& a, hipStream_t s) {
  dim3 grid((unsigned)(a.BH * a.T)), block(DQ_NT);
  auto kernel = dq_kernel<E, D, 0>;
  if (a.gk == 1) kernel = dq_kernel<E, D, 1>;
  if (a.gk == 2) kernel = dq_kernel<E, D, 2>;
  if (a.gk == 4) kernel = dq_kernel<E, D, 4>;
  return launch_kernel(kernel, grid, block, s, a);
}

template <typename E, int D>
hipError_t launch_collect_d(const CollectArgs& a, hipStream_t s) {
  if constexpr (sizeof(E) == 2) {
    const dim3 sampled((unsigned)(a.BH * sampled_blocks(a.T)));
    const hipError_t e = launch_kernel(probe_kernel<E, D>, sampled, dim3(COL_NT), s, a);
    if (e != hipSuccess) return e;
  }
  dim3 grid((unsigned)(a.BH * ((a.T + 1) / 2))), block(COL_NT);
  auto kernel = collect_kernel<E, D, 1>;  // the kinds but fp32's general alpha differ in nothing here
  if (sizeof(E) == 4 && a.gk == 0) kernel = collect_kernel<E, D, 0>;
  return launch_kernel(kernel, grid, block, s, a);
}

template <typename E, int D>
hipError_t launch_dkdv_lists_d(const BwdArgs& a, hipStream_t s) {
  dim3 grid((unsigned)(a.BH * a.T)), block(LK_NT);
  auto kernel = dkdv_lists_kernel<E, D, 0>;
  if (a.gk == 1) kernel = dkdv_lists_kernel<E, D, 1>;
  if (a.gk == 2) kernel = dkdv_lists_kernel<E, D, 2>;
  if (a.gk == 4) kernel = dkdv_lists_kernel<E, D, 4>;
  return launch_kernel(kernel, grid, block, s, a);
}

template <typename E, int D>
hipError_t launch_delta_d(const DeltaArgs& a, hipStream_t s) {
  if (a.lists) return launch_kernel(prep_kernel<E, D>, dim3((unsigned)(a.BH * a.T)), dim3(PREP_NT), s, a);
  dim3 grid((unsigned)((a.rows + 15) / 16)), block(256);
  return launch_kernel(delta_kernel<E, D>, grid, block, s, a);
}

}  // namespace

hipError_t launch_delta(const DeltaArgs& a, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0) return head_dim == 64 ? launch_delta_d<__bf16, 64>(a, s) : launch_delta_d<__bf16, 128>(a, s);
  return head_dim == 64 ? launch_delta_d<float, 64>(a, s) : launch_delta_d<float, 128>(a, s);
}

hipError_t launch_bwd_dkdv(const BwdArgs& a, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0) return head_dim == 64 ? launch_dkdv_d<__bf16, 64>(a, s) : launch_dkdv_d<__bf16, 128>(a, s);
  return head_dim == 64 ? launch_dkdv_d<float, 64>(a, s) : launch_dkdv_d<float, 128>(a, s);
}

hipError_t launch_collect(const CollectArgs& a, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0) return head_dim == 64 ? launch_collect_d<__bf16, 64>(a, s) : launch_collect_d<__bf16, 128>(a, s);
  return head_dim == 64 ? launch_collect_d<float, 64>(a, s) : launch_collect_d<float, 128>(a, s);
}

hipError_t launch_bwd_dkdv_lists(const BwdArgs& a, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0)
    return head_dim == 64 ? launch_dkdv_lists_d<__bf16, 64>(a, s) : launch_dkdv_lists_d<__bf16, 128>(a, s);
  return head_dim == 64 ? launch_dkdv_lists_d<float, 64>(a, s) : launch_dkdv_lists_d<float, 128>(a, s);
}

hipError_t launch_bwd_dq(const BwdArgs& a, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0) return head_dim == 64 ? launch_dq_d<__bf16, 64>(a, s) : launch_dq_d<__bf16, 128>(a, s);
  return head_dim == 64 ? launch_dq_d<float, 64>(a, s) : launch_dq_d<float, 128>(a, s);
}

}  // namespace ea
