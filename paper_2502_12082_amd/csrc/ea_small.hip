// ea_small.hip -- the threshold solver for short sequences (n <= 1024).
//
// The same method and rules as solve_kernel (ea_tau.hip): pass 0 with the
// bracket's lower end from the largest scores of distinct keys, Algorithm 1 on
// the scores above it, the mask, row table and element lists at the returned
// tau.  But a row this short needs no candidate cache in memory: one workgroup
// of 8 waves owns a 64-row query block, wave (rg, kg) scores the 32 rows rg
// against every fourth 32-key tile, and keeps all of those scores in
// registers (16 per tile and lane).  The scores above the lower end go to
// short lists in LDS, one per lane, on which the evaluations run; the eight
// lanes of a row add their sums up through LDS.  K is read once, straight into
// the A operands.
//
// What bounds it is the latency of that chain, not a rate: the cached solver
// took 45-50 us for n = 256 ... 777 whatever the grid (its lists are written
// to and read back from L2 in every step), and 110 us on B8 H12 n1024 d64.
#include <type_traits>

#include "ea_common.h"
#include "ea_internal.h"

namespace ea {

namespace {

constexpr int SM_NT = 512;
constexpr int SM_KG = 4;      // key groups (waves per row group)
constexpr int SM_LIST = 16;   // entries of a lane's list

// Columns 8 m .. 8 m + 7 of a fp32 row, held as 8 m + 4 h + e by the row's two
// lanes (h = lane half), as the operands of the four products that take them:
// step e has columns 8 m + 2 e + h (see load_row_frag_global).  The products
// are then added up in the order of every other kernel, so that the scores,
// and with them the mask and the support at tau, are theirs bit for bit.
__device__ __forceinline__ f32x4 step_operands(const f32x4& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2]), __float_as_uint(v[3]), false, false);
  return f32x4{__uint_as_float(a[0]), __uint_as_float(b[0]), __uint_as_float(a[1]), __uint_as_float(b[1])};
#else
  return v;
#endif
}

template <typename E, int D, int GK, int KT>
__global__ __launch_bounds__(SM_NT, KT <= 4 ? 4 : 2) void solve_small_kernel(TauArgs a) {
  using M = Mma<E>;
  constexpr int KS = D / M::KW;
  __shared__ float list[SM_LIST + 1][SM_NT];  // the last row takes dropped stores
  __shared__ __attribute__((aligned(16))) f32x4 part[SM_KG][BLK];  // sums; first the largest scores
  __shared__ int count[SM_KG][2][64];
  __shared__ uint32_t bits;
  __shared__ int over, entries;

  const int t = threadIdx.x, lane = lane_id(), w = wave_id(), rg = w & 1, kg = w >> 1, half = lane >> 5;
  const int n = a.n, T = a.T;
  const int bh = blockIdx.x % a.BH, qb = blockIdx.x / a.BH;
  const int q0 = qb * BLK + 32 * rg, i = q0 + (lane & 31), row = 32 * rg + (lane & 31);
  const bool row_ok = i < n;
  const float c = a.c, g = a.gamma;
  const bool newton_bound = g >= 1.f;
  const E* Q = static_cast<const E*>(a.q) + (size_t)bh * n * D;
  const E* K = static_cast<const E*>(a.k) + (size_t)bh * n * D;
  const int keys = a.causal ? min(n, q0 + 32) : n;  // keys any row of the wave sees
  if (t == 0) {
    bits = 0;
    over = 0;
    entries = 0;
  }

  // ---- scores: value r of tile k is key 32 (kg + 4 k) + crow(r), row lane % 32
  f32x16 s[KT];
  if constexpr (sizeof(E) == 2) {
    typename M::frag qf[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = load_row_frag_global<E, D>(Q, i, n, kk);
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      s[k] = zero16();
      const int j0 = 32 * (kg + SM_KG * k);
      if (j0 < keys && q0 < n) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk)
          s[k] = M::mma(load_row_frag_global<E, D>(K, min(j0 + (lane & 31), n - 1), n, kk), qf[kk], s[k]);
      }
    }
  } else {
    // fp32: 16-byte loads, then four operands (Q's in the first tile, so that
    // its keys are on the way meanwhile; a wave without that tile has no other)
    f32x4 qf[D / 8];
    const float* qr = reinterpret_cast<const float*>(Q) + (size_t)min(i, n - 1) * D + 4 * half;
#pragma unroll
    for (int m = 0; m < D / 8; ++m) qf[m] = *reinterpret_cast<const f32x4*>(qr + 8 * m);
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      s[k] = zero16();
      const int j0 = 32 * (kg + SM_KG * k);
      if (j0 < keys && q0 < n) {
        const float* kr = reinterpret_cast<const float*>(K) + (size_t)min(j0 + (lane & 31), n - 1) * D + 4 * half;
#pragma unroll
        for (int m = 0; m < D / 8; ++m) {
          const f32x4 kf = step_operands(*reinterpret_cast<const f32x4*>(kr + 8 * m));
          if (k == 0) qf[m] = step_operands(qf[m]);
#pragma unroll
          for (int e = 0; e < 4; ++e) s[k] = M::mma(kf[e], qf[m][e], s[k]);
        }
      }
    }
  }
  // invalid pairs become -inf: never a maximum, and z = 0
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    const int j0 = 32 * (kg + SM_KG * k);
    if (j0 + 31 >= n || (a.causal && j0 + 31 > q0) || q0 + 31 >= n) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int j = j0 + crow(r);
        if (!(row_ok && j < n && (!a.causal || j <= i))) s[k][r] = -INFINITY;
      }
    }
  }

  // ---- pass 0: each lane's two largest tile maxima (distinct keys), sixteen
  // values per row; their own root by Newton steps from below is a lower
  // bound of tau (f restricted to these keys is convex, decreasing and no
  // larger than f)
  float m1 = -INFINITY, m2 = -INFINITY;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    float v = max3f(s[k][0], s[k][1], s[k][2]);
#pragma unroll
    for (int r = 3; r < 15; r += 2) v = max3f(v, s[k][r], s[k][r + 1]);
    v = fmaxf(v, s[k][15]);
    m2 = fmaxf(m2, fminf(m1, v));
    m1 = fmaxf(m1, v);
  }
  {
    float lo1, hi1, lo2, hi2;
    wave_halves(m1, lo1, hi1);
    wave_halves(m2, lo2, hi2);
    if (half == 0) part[kg][row] = f32x4{lo1, hi1, lo2, hi2};
  }
  __syncthreads();
  float lo = 0.f, hi = 0.f, tau = 0.f;
  {
    float u[16];
#pragma unroll
    for (int x = 0; x < SM_KG; ++x) {
      const f32x4 v = part[x][row];
#pragma unroll
      for (int e = 0; e < 4; ++e) u[4 * x + e] = v[e];
    }
    if (row_ok) {
      float m = u[0];
#pragma unroll
      for (int x = 1; x < 16; ++x) m = fmaxf(m, u[x]);
      m *= c;
      const float ni = (float)(a.causal ? i + 1 : n);
      hi = m - powf(ni, 1.f - a.alpha);
      float b = m - 1.f;
      if (newton_bound) {
#pragma unroll 1
        for (int it = 0; it < 3; ++it) {
          float f = -1.f, fp = 0.f;
#pragma unroll
          for (int x = 0; x < 16; ++x) {
            float pj, uj;
            Gamma<GK>::pu(relu_z(c, u[x], b), g, pj, uj);
            f += pj;
            fp += uj;
          }
          if (f > 0.f) b += f / (g * fp);
        }
      } else {
        // f is not convex: one term of f at a time (solve_kernel's bound):
        // with j scores at or above u_x, j (c u_x - tau)^gamma <= 1
#pragma unroll 1
        for (int x = 0; x < 16; ++x) {
          const float ux = part[x >> 2][row][x & 3];
          int j = 0;
#pragma unroll
          for (int y = 0; y < 16; ++y) j += u[y] >= ux ? 1 : 0;
          if (ux > -INFINITY) b = fmaxf(b, fmaf(c, ux, -exp2f(-__log2f((float)j) / g)));
        }
      }
      lo = fminf(b - 4e-6f * fmaxf(1.f, fabsf(b)), hi);
      tau = newton_bound ? fminf(b, hi) : 0.5f * (lo + hi);
    }
  }

  // ---- this lane's scores above the lower end (less a margin for the
  // rounding of lo / c): to its list, and a bit per score in `cand`
  const float t0 = lo / c;
  const float s_lo = row_ok ? t0 - 1e-6f * fmaxf(fabsf(t0), 1.f / c) : INFINITY;
  uint32_t cand[(KT + 1) / 2];  // bit 16 (k % 2) + r of word k / 2
  int cc = 0;
#pragma unroll
  for (int x = 0; x < (KT + 1) / 2; ++x) cand[x] = 0;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    if (32 * (kg + SM_KG * k) >= keys) break;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const bool in = s[k][r] > s_lo;
      list[min(cc, SM_LIST)][t] = s[k][r];
      cand[k / 2] |= in ? 1u << (16 * (k & 1) + r) : 0u;
      cc += in ? 1 : 0;
    }
  }
  if (__ballot(cc > SM_LIST) != 0ull && lane == 0) over = 1;
  __syncthreads();  // `part` has been read, too
  const bool listed = over == 0;
  int cmax = cc;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) cmax = max(cmax, __shfl_xor(cmax, o));

  // ---- Algorithm 1
  int evals = 0;
  float f_prev = INFINITY;
  for (int it = 0;; ++it) {
    float v0 = 0.f, v1 = 0.f, v2 = 0.f;
    auto add = [&](float zp) {
      if constexpr (GK == 1) {
        v0 += zp;
        v1 += zp > 0.f ? 1.f : 0.f;
      } else if constexpr (GK == 2) {
        v0 = fmaf(zp, zp, v0);
        v1 += zp;
        v2 += zp > 0.f ? 1.f : 0.f;
      } else if constexpr (GK == 4) {
        const float z2 = zp * zp;
        v0 = fmaf(z2, z2, v0);
        v1 = fmaf(z2, zp, v1);
        v2 += z2;
      } else if (zp > 0.f) {
        const float l = __log2f(zp);
        v0 += exp2f(g * l);
        v1 += exp2f((g - 1.f) * l);
        v2 += exp2f((g - 2.f) * l);
      }
    };
    if (listed) {
      for (int e0 = 0; e0 < cmax; e0 += 4) {
        float x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = list[min(e0 + u, SM_LIST)][t];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (e0 + u < cc) add(relu_z(c, x[u], tau));
      }
    } else {
#pragma unroll
      for (int k = 0; k < KT; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) add(relu_z(c, s[k][r], tau));
    }
    v0 = sum_halves(v0);
    v1 = sum_halves(v1);
    v2 = sum_halves(v2);
    if (half == 0) part[kg][row] = f32x4{v0, v1, v2, 0.f};
    __syncthreads();
    f32x4 sum = part[0][row];
#pragma unroll
    for (int x = 1; x < SM_KG; ++x) sum += part[x][row];
    const float f = sum[0] - 1.f;  // Eq. 3
    float f1, f2;                  // Eq. 6, 7
    if constexpr (GK == 1) {
      f1 = -sum[1];
      f2 = 0.f;
    } else if constexpr (GK == 2) {
      f1 = -2.f * sum[1];
      f2 = 2.f * sum[2];
    } else if constexpr (GK == 4) {
      f1 = -4.f * sum[1];
      f2 = 12.f * sum[2];
    } else {
      f1 = -g * sum[1];
      f2 = g * (g - 1.f) * sum[2];
    }
    const bool conv = !row_ok || fabsf(f) <= a.tol;
    const bool stop = __syncthreads_and(conv) || it >= a.max_iter;
    evals = it + 1;
    if (row_ok) {
      // the update rules of solve_kernel; the last evaluation's update is
      // taken as well (the mask is built afterwards)
      if (f < 0.f)
        hi = tau;
      else
        lo = tau;
      const float slack = 1e-6f * fmaxf(1.f, fmaxf(fabsf(lo), fabsf(hi)));
      if (newton_bound && f1 < 0.f) lo = fminf(fmaxf(lo, tau - f / f1 - 10.f * slack), hi);
      const float th = tau - 2.f * f * f1 / (2.f * f1 * f1 - f * f2);
      bool take = th >= lo - slack && th <= hi + slack;
      if (!newton_bound && fabsf(f) > 0.5f * f_prev) take = false;
      f_prev = fabsf(f);
      // (below a bracket whose lower end is Newton's bound: that end is the
      // better guess)
      tau = take ? fminf(fmaxf(th, lo), hi) : newton_bound && th < lo ? lo : 0.5f * (lo + hi);
    }
    if (stop) break;
  }

  if (row_ok && half == 0 && kg == 0) {
    a.tau[(size_t)bh * n + i] = tau;
    if (std::is_same<E, float>::value) a.tau_lo[(size_t)bh * n + i] = 0.f;
  }

  // ---- mask bits, and the element lists: the lists of a row's two halves
  // hold the entries of its four waves one after another
  uint32_t tiles = 0;  // bit k: a positive probability in tile k (uniform)
  int mine = 0;
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    if (32 * (kg + SM_KG * k) >= keys) break;
    int in = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) in += in_support(relu_z(c, s[k][r], tau));
    mine += in;
    if (__ballot(in > 0) != 0ull) tiles |= 1u << k;
  }
  count[kg][rg][lane] = mine;
  int total = mine;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) total += __shfl_xor(total, o);
  if (lane == 0) {
    uint32_t b = 0;
#pragma unroll
    for (int k = 0; k < KT; ++k)
      if (tiles >> k & 1u) b |= 1u << ((kg + SM_KG * k) >> 1);
    atomicOr(&bits, b);
    atomicAdd(&entries, total);
  }
  __syncthreads();
  const uint32_t mask = bits;
  const int blocks = __popc(mask);
  ListBlock* const lb = a.lists ? a.lists + ((size_t)bh * T + qb) : nullptr;
  const int use = list_use(entries, blocks, T, sizeof(E) == 4);
  bool fit = listed && use != LIST_NONE;
  int base = 0, all = 0;
#pragma unroll
  for (int x = 0; x < SM_KG; ++x) {
    if (x < kg) base += count[x][rg][lane];
    all += count[x][rg][lane];
  }
  fit = __syncthreads_and(fit && all <= LIST_CAP);
  if (lb) {
    if (fit) {
      // candidate e of this lane is the e-th set bit of `cand`
      const int id = 64 * half + row;
      int at = LIST_IDS * base + id, e = 0;
#pragma unroll
      for (int x = 0; x < (KT + 1) / 2; ++x) {
        uint32_t m = cand[x];
        while (__ballot(m != 0) != 0ull) {
          if (m != 0) {
            const int b = __ffs(m) - 1;
            m &= m - 1;
            const float zp = relu_z(c, list[e][t], tau);
            ++e;
            if (zp > 0.f) {
              const int r = b & 15, k = 2 * x + (b >> 4);
              lb->z[at] = zp;
              lb->key[at] = (uint16_t)(32 * (kg + SM_KG * k) + 8 * (r >> 2) + 4 * half + (r & 3));
              at += LIST_IDS;
            }
          }
        }
      }
      if (kg == 0) {
        lb->count[id] = (uint8_t)all;
        if (half == 0 && row_ok) lb->tau[row] = tau;
      }
    }
    if (t == 0) a.use[(size_t)bh * T + qb] = fit ? use : LIST_NONE;
  }
  if (w != 0) return;
  // mask row and row table (at most 16 key blocks)
  const bool b = lane < T && (mask >> lane & 1u), tables = a.mask != nullptr;
  if (tables && lane < T) a.mask[((size_t)bh * T + qb) * T + lane] = b ? 1 : 0;
  const unsigned long long m = __ballot(b);
  if (tables && b) a.q_index[((size_t)bh * T + qb) * T + __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)] = lane;
  if (lane == 0) {
    if (tables) a.q_count[(size_t)bh * T + qb] = blocks;
    if (a.stats) {
      a.stats[(size_t)bh * T + qb] = 1;
      a.stats[((size_t)a.BH + bh) * T + qb] = evals;
    }
  }
}

template <typename E, int D, int GK>
hipError_t launch_small_g(const TauArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)(a.BH * a.T)), block(SM_NT);
  if (a.n <= 256) return launch_kernel(solve_small_kernel<E, D, GK, 2>, grid, block, s, a);
  if (a.n <= 512) return launch_kernel(solve_small_kernel<E, D, GK, 4>, grid, block, s, a);
  return launch_kernel(solve_small_kernel<E, D, GK, 8>, grid, block, s, a);
}

template <typename E, int D>
hipError_t launch_small_d(const TauArgs& a, hipStream_t s) {
  if (a.gk == 1) return launch_small_g<E, D, 1>(a, s);
  if (a.gk == 2) return launch_small_g<E, D, 2>(a, s);
  if (a.gk == 4) return launch_small_g<E, D, 4>(a, s);
  if constexpr (sizeof(E) == 2) return launch_small_g<E, D, 0>(a, s);
  return hipErrorInvalidValue;  // (fp32 inputs with a general alpha: solve_kernel)
}

}  // namespace

hipError_t launch_tau_small(const TauArgs& a, int dtype, int head_dim, hipStream_t s) {
  if (dtype == 0)
    return head_dim == 64 ? launch_small_d<__bf16, 64>(a, s) : launch_small_d<__bf16, 128>(a, s);
  return head_dim == 64 ? launch_small_d<float, 64>(a, s) : launch_small_d<float, 128>(a, s);
}

}  // namespace ea
