// What consumes the scores: per-segment top-K (the inference phase of
// section 3 keeps the K best candidates of a tuning round) and the RDU
// sampler's selection of programs to label (section 4, Alg. 1, Eq. (1)-(3)).
//
// Top-K: one workgroup of 1,024 threads per segment. Scores map to
// order-preserving 32-bit keys (NaN below everything); a radix select finds a
// key that at least K and not many more keys reach, and those are gathered and
// ranked in LDS by (key descending, index ascending). Where too many keys
// equal the K-th, the lowest-index ones are taken.
//
// RDU selection: the greedy loop of Alg. 1, one launch per selected program
// (the host only enqueues), over the whole pool or over the short list of
// candidates that can win: see rdu_score_kernel. A candidate
// whose operator type has used its budget can never be labeled, so it is
// masked out as soon as that is seen; Alg. 1 drops such candidates one at a
// time when they come up as the argmax, which leaves the same sequence of
// labeled programs. fp64 throughout (the normalised predictions, distances,
// sums and t_s).
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace tcl {
namespace {

constexpr int kST = 256;  // threads per block

// ---------------------------------------------------------------- top-K
__device__ __forceinline__ uint32_t score_key(float f) {
  if (f != f) return 0u;  // NaN: below every number
  uint32_t u = __float_as_uint(f);
  if ((u << 1) == 0u) u = 0u;  // -0 and +0 are equal scores
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kTK = 1024;  // threads of a top-K workgroup

// block-wide exclusive prefix of a 0/1 flag over the kTK threads (in thread
// order); returns the prefix, *total the block's count
__device__ __forceinline__ int block_prefix(bool flag, int* wsum, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t m = __ballot(flag);
  const int in_wave = __popcll(m & ((1ull << lane) - 1ull));
  __syncthreads();
  if (lane == 0) wsum[w] = __popcll(m);
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kTK / 64; ++i) {
    before += i < w ? wsum[i] : 0;
    all += wsum[i];
  }
  *total = all;
  return before + in_wave;
}

// CAP: candidates gathered at most, >= K. Digits of 12, 10 and 10 bits, the
// first alone when the K-th key's bin is short: with 4,096 scores and K = 64 it
// holds some 60 keys (an eighth of a power of two), and what lies above and in
// it fits the candidates. Each candidate's place is then the number of larger
// ones. Up to kTKeys keys a thread stay in registers. Two workgroups fit on a
// CU (at most 64 VGPRs and 100 SGPRs), for calls of more segments than CUs, and
// keys that share a bin are counted without 64 lanes queueing for one address.
// Calls back to back with the scores in cache, K = 64, against four 8-bit passes over
// memory and a bitonic sort: 16 segments of 4,096 14.3 -> 8.1 us (a launch, one round of
// loads and a dozen barriers), of equal scores 25.1 -> 14.3; one of 65,536 108 -> 21.
// 300 segments of 600 with equal scores, K = 10: 14.6 -> 11.0 (19.1 with one workgroup
// a CU and one atomic a key).
constexpr int kTKeys = 8;
template <int CAP>
__global__ __launch_bounds__(kTK, 8) void topk_kernel(const int* __restrict__ offs, const float* __restrict__ s,
                                                   int K, int* __restrict__ out) {
  constexpr int kBins = 4096;
  static_assert(kBins == 4 * kTK, "four counters a thread");
  __shared__ __attribute__((aligned(16))) uint64_t cand[CAP];
  __shared__ __attribute__((aligned(16))) int hist[kBins];
  __shared__ int tot[kTK / 64];
  __shared__ int wsum[kTK / 64];
  __shared__ int sdig, sabove, scount, cnt;
  const int g = blockIdx.x;
  const int lo = offs[g];
  const int n = max(offs[g + 1] - lo, 0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int take = min(n, K);

  const bool regs = n <= kTKeys * kTK;  // block-uniform
  uint32_t key[kTKeys];
  if (regs) {
#pragma unroll
    for (int r = 0; r < kTKeys; ++r) key[r] = n > 0 ? score_key(s[lo + min(tid + r * kTK, n - 1)]) : 0u;
  }
  // f(key, index) of every key of this thread
  auto visit = [&](auto f) {
    if (regs) {
#pragma unroll
      for (int r = 0; r < kTKeys; ++r)
        if (tid + r * kTK < n) f(key[r], tid + r * kTK);
    } else {
      for (int i0 = tid; i0 < n; i0 += kTKeys * kTK) {  // a round's loads together
        float v[kTKeys];
#pragma unroll
        for (int r = 0; r < kTKeys; ++r) v[r] = s[lo + min(i0 + r * kTK, n - 1)];
#pragma unroll
        for (int r = 0; r < kTKeys; ++r)
          if (i0 + r * kTK < n) f(score_key(v[r]), i0 + r * kTK);
      }
    }
  };
  auto code_of = [](uint32_t k, int i) { return ((uint64_t)k << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)i); };

  if (tid == 0) cnt = 0;
  uint32_t least = 0u;  // candidates: keys >= least
  bool exact = true;    // they fit CAP
  int krem = K;
  if (n > K) {
    uint32_t prefix = 0u, pmask = 0u;
    int above = 0;
    exact = false;
    auto digit = [&](auto PASS) {
      constexpr int pass = decltype(PASS)::value, shift = pass == 0 ? 20 : pass == 1 ? 10 : 0;
      reinterpret_cast<int4*>(hist)[tid] = int4{0, 0, 0, 0};
      __syncthreads();
      visit([&](uint32_t k, int i) {
        if ((k & pmask) != prefix) return;
        const int bin = pass == 0 ? (int)(k >> 20) : 4 * ((int)(k >> shift) & 1023) + (lane & 3);
        // close scores share a few bins, where 64 lanes would queue for one
        // address: a short segment's lanes in the first one's bin count together
        if (pass == 0 && regs && i < kTK) {
          const int first = __builtin_amdgcn_readfirstlane(bin);
          const uint64_t same = __builtin_amdgcn_ballot_w64(bin == first);
          if (bin != first) atomicAdd(&hist[bin], 1);
          else if (lane == __builtin_ctzll(same)) atomicAdd(&hist[bin], __builtin_popcountll(same));
        } else {
          atomicAdd(&hist[bin], 1);
        }
      });
      __syncthreads();
      // thread t takes four counters from 4095 - 4 t down: four digits, or the
      // four parts of one, by lane, that the later digits are counted in (one atomic in
      // four to an address). A scan over threads gives the count of keys at or above
      // each digit, and exactly one has that count reach krem while the digits
      // above it stay below
      const int4 h = reinterpret_cast<const int4*>(hist)[kTK - 1 - tid];
      const int c[4] = {pass == 0 ? h.w : h.x + h.y + h.z + h.w, pass == 0 ? h.z : 0, pass == 0 ? h.y : 0,
                        pass == 0 ? h.x : 0};
      const int sum = c[0] + c[1] + c[2] + c[3];
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
      }
      if (lane == 63) tot[wave] = incl;
      __syncthreads();
      int at = incl - sum;
#pragma unroll
      for (int w = 0; w < kTK / 64; ++w) at += w < wave ? tot[w] : 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (at < krem && at + c[r] >= krem) {
          sdig = pass == 0 ? kBins - 1 - (4 * tid + r) : kTK - 1 - tid;
          sabove = at;
          scount = c[r];
        }
        at += c[r];
      }
      __syncthreads();
      krem -= sabove;
      above += sabove;
      prefix |= (uint32_t)sdig << shift;
      pmask |= (pass == 0 ? 0xFFFu : 0x3FFu) << shift;
      least = prefix;
      exact = above + scount <= CAP;
    };
    digit(std::integral_constant<int, 0>{});
    if (!exact) digit(std::integral_constant<int, 1>{});
    if (!exact) digit(std::integral_constant<int, 2>{});
  }
  __syncthreads();
  if (exact) {
    visit([&](uint32_t k, int i) {
      if (k >= least) cand[atomicAdd(&cnt, 1)] = code_of(k, i);
    });
    __syncthreads();
  } else {
    // more keys equal to the K-th than fit: those above it, then the first
    // krem equal ones in index order
    int eq_base = 0;
    for (int t0 = 0; t0 < n; t0 += kTK) {
      const int i = t0 + tid;
      const bool ok = i < n;
      const uint32_t k = ok ? score_key(s[lo + i]) : 0u;
      if (ok && k > least) cand[atomicAdd(&cnt, 1)] = code_of(k, i);
      const bool eq = ok && k == least;
      int all;
      const int r = block_prefix(eq, wsum, &all);
      if (eq && eq_base + r < krem) cand[(take - krem) + eq_base + r] = code_of(k, i);
      eq_base += all;
    }
    __syncthreads();
    if (tid == 0) cnt = take;
    __syncthreads();
  }
  const int m = cnt;
  for (int i = tid; i < m; i += kTK) {
    const uint64_t mine = cand[i];
    int rank = 0, q = 0;
#pragma unroll 4
    for (; q + 1 < m; q += 2) {
      const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(&cand[q]);
      rank += (v.x > mine) + (v.y > mine);
    }
    if (q < m) rank += cand[q] > mine;
    if (rank < take) out[(int64_t)g * K + rank] = lo + (int)(0xFFFFFFFFu - (uint32_t)(mine & 0xFFFFFFFFull));
  }
  for (int r = take + tid; r < K; r += kTK) out[(int64_t)g * K + r] = -1;
}

// ---------------------------------------------------------------- RDU selection
struct RduState {
  double lo, range;  // normalisation of the predictions
  double S1, S2;     // sums of f and f^2 over the labeled set
  int M;             // labeled programs
  int count;         // selected so far
  int last;          // the last selected program (-1: none yet)
  int done;
  int n_select;
  unsigned arrived;  // blocks of the current launch that have parked their partial
  int ver;           // labeled programs the whole pool's distances include
  int nact;          // candidates collected for the short list
  int mode[2];       // what a launch of this parity does: RduMode
  int collect;       // this launch, over the whole pool, collects those with t_s >= cut
  int spare;         // launches that may still come to nothing
  double cut;            // the short list's bound
  double cut_S1, cut_S2; // S1, S2 and M when it was collected
  int cut_M;
  int run;               // selections made from it
  int balance, cost;     // selections that lists served, less the cost of each try at one
  int wait, back, back0; // kRduPlain launches until the next try, and how many the time after
  double next_cut;       // the bound the last pass over the whole pool suggests
};

enum RduMode {
  kRduWhole,  // over the whole pool, with every label since the last such launch; may sample and collect
  kRduListed, // over the short list
  kRduPlain,  // over the whole pool, with the last label
};

struct Best {
  double t;
  int i;
};

__device__ __forceinline__ bool better(double t, int i, double bt, int bi) {
  return bi < 0 || t > bt || (t == bt && i < bi);
}

__device__ __forceinline__ double fhat(const float* s, int i, const RduState& st) {
  return st.range > 0.0 ? ((double)s[i] - st.lo) / st.range : 0.0;
}

// per block: min and max of the scores, and a histogram of operator types
// (types outside [0, n_ops) are counted in opcount[n_ops])
constexpr int kMaxOps = 4096;
__global__ __launch_bounds__(kST) void rdu_stats_kernel(int N, const float* __restrict__ s,
                                                        const int* __restrict__ op, int n_ops,
                                                        float* __restrict__ mm, int* __restrict__ opcount) {
  __shared__ float smin[kST], smax[kST];
  __shared__ int h[kMaxOps + 1];
  for (int o = threadIdx.x; o <= n_ops; o += kST) h[o] = 0;
  __syncthreads();
  float mn = INFINITY, mx = -INFINITY;
  for (int i = blockIdx.x * kST + threadIdx.x; i < N; i += gridDim.x * kST) {
    mn = fminf(mn, s[i]);
    mx = fmaxf(mx, s[i]);
    const int o = op[i];
    atomicAdd(&h[(o >= 0 && o < n_ops) ? o : n_ops], 1);
  }
  __syncthreads();
  for (int o = threadIdx.x; o <= n_ops; o += kST)
    if (h[o]) atomicAdd(&opcount[o], h[o]);
  smin[threadIdx.x] = mn;
  smax[threadIdx.x] = mx;
  __syncthreads();
  for (int o = kST / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      smin[threadIdx.x] = fminf(smin[threadIdx.x], smin[threadIdx.x + o]);
      smax[threadIdx.x] = fmaxf(smax[threadIdx.x], smax[threadIdx.x + o]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    mm[2 * blockIdx.x] = smin[0];
    mm[2 * blockIdx.x + 1] = smax[0];
  }
}

__global__ __launch_bounds__(kST) void rdu_zero_kernel(int n, int* __restrict__ a) {
  for (int i = blockIdx.x * kST + threadIdx.x; i < n; i += gridDim.x * kST) a[i] = 0;
}

// Histogram, over a sample of the pool, of how far t_s is above the smallest
// u_s: bins of an eighth of a power of two, from 2^-40 up.
constexpr int kHistBins = 42 * 8, kHistFirst = (1023 - 40) * 8;
constexpr int kHistEvery = 32;  // one candidate in so many: one of four in every eighth block
__device__ __forceinline__ int hist_bin(double t) {
  const int b = (int)((uint64_t)__double_as_longlong(t) >> 49) - kHistFirst;
  return t > 0.0 ? max(0, min(b, kHistBins - 1)) : 0;
}
__device__ __forceinline__ double u_min(double S1, double S2, double inv) {
  // u = (inv - inv^2) f^2 - 2 S1 inv^2 f + S2 inv - (S1 inv)^2, f in [0, 1]
  const double a = inv - inv * inv, f = a > 0.0 ? fmin(S1 * inv * inv / a, 1.0) : 1.0;
  const double mu = (f + S1) * inv;
  return (f * f + S2) * inv - mu * mu;
}
__device__ __forceinline__ double hist_edge(int b) {
  return __longlong_as_double((long long)((uint64_t)(b + kHistFirst) << 49));
}

// one block: normalisation, budgets, sums over the initial labeled set
__global__ __launch_bounds__(kST) void rdu_setup_kernel(int N, const float* __restrict__ s, int n_ops,
                                                        const int* __restrict__ init, int n_init, int n_select,
                                                        const float* __restrict__ mm, int nmm,
                                                        const int* __restrict__ opcount,
                                                        double* __restrict__ budget, int* __restrict__ sel,
                                                        int spare, int* __restrict__ hist,
                                                        RduState* __restrict__ state) {
  __shared__ double r1[kST], r2[kST];
  __shared__ int rc[kST];
  __shared__ float smn[kST], smx[kST];
  {
    float mn = INFINITY, mx = -INFINITY;
    for (int b = threadIdx.x; b < nmm; b += kST) {
      mn = fminf(mn, mm[2 * b]);
      mx = fmaxf(mx, mm[2 * b + 1]);
    }
    smn[threadIdx.x] = mn;
    smx[threadIdx.x] = mx;
  }
  __syncthreads();
  for (int o = kST / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      smn[threadIdx.x] = fminf(smn[threadIdx.x], smn[threadIdx.x + o]);
      smx[threadIdx.x] = fmaxf(smx[threadIdx.x], smx[threadIdx.x + o]);
    }
    __syncthreads();
  }
  RduState st{};
  st.lo = (double)smn[0];
  st.range = (double)smx[0] - (double)smn[0];
  for (int o = threadIdx.x; o < n_ops; o += kST) {
    budget[o] = (double)n_select * (double)opcount[o] / (double)N;
    sel[o] = 0;
  }
  if (hist) {
    for (int o = threadIdx.x; o < kHistBins; o += kST) hist[o] = 0;
  }
  double a1 = 0.0, a2 = 0.0;
  int c = 0;
  for (int j = threadIdx.x; j < n_init; j += kST) {
    const int i = init[j];
    if (i >= 0 && i < N) {
      const double f = fhat(s, i, st);
      a1 += f;
      a2 += f * f;
      ++c;
    }
  }
  r1[threadIdx.x] = a1;
  r2[threadIdx.x] = a2;
  rc[threadIdx.x] = c;
  __syncthreads();
  for (int o = kST / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      r1[threadIdx.x] += r1[threadIdx.x + o];
      r2[threadIdx.x] += r2[threadIdx.x + o];
      rc[threadIdx.x] += rc[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    st.S1 = r1[0];
    st.S2 = r2[0];
    st.M = rc[0];
    st.count = 0;
    st.last = -1;
    st.n_select = n_select;
    st.done = (n_select <= 0 || rc[0] == 0) ? 1 : 0;
    st.spare = spare;
    // measured over 140,000 to 8.65 M programs, 8 to 512 selections of equal,
    // tied, log-normal, normal and sorted scores: half of this cost is within 2 %,
    // twice as much loses up to 9 %, four times up to half; without a wait 2.6
    // times the call (64 different scores, 8.65 M, 512 selections), waiting for
    // good 2.3 times (normal scores there)
    st.balance = st.cost = N < 524288 ? 4 : 1;
    st.back = st.back0 = N < 524288 ? 32 : 8;
    *state = st;
  }
}

// The initial labeled set's normalised predictions, sorted ascending (at
// most kSortInit of them; larger sets use rdu_dinit_kernel's direct pass).
constexpr int kSortInit = 8192;
__global__ __launch_bounds__(1024) void rdu_sort_init_kernel(int N, const float* __restrict__ s,
                                                             const int* __restrict__ init, int n_init,
                                                             const RduState* __restrict__ state,
                                                             double* __restrict__ sorted, int* __restrict__ n_valid) {
  __shared__ double v[kSortInit];
  const RduState st = *state;
  int P = 1;
  while (P < n_init) P <<= 1;
  for (int j = threadIdx.x; j < P; j += 1024) {
    const int i = j < n_init ? init[j] : -1;
    v[j] = (i >= 0 && i < N && s[i] == s[i]) ? fhat(s, i, st) : INFINITY;  // invalid entries sort last
  }
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1) {
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
      for (int i = threadIdx.x; i < P; i += 1024) {
        const int p = i ^ jj;
        if (p > i) {
          const double a = v[i], b = v[p];
          const bool up = (i & k) == 0;
          if (up ? (a > b) : (a < b)) {
            v[i] = b;
            v[p] = a;
          }
        }
      }
      __syncthreads();
    }
  }
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int j = threadIdx.x; j < n_init; j += 1024) {
    sorted[j] = v[j];
    if (v[j] != INFINITY) atomicAdd(&cnt, 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) *n_valid = cnt;
}

// d[i] = min over the initial set of |f_i - f_j|: the nearest value on each
// side of f_i in the sorted set (a binary search) gives the same minimum
__global__ __launch_bounds__(kST) void rdu_dinit_sorted_kernel(int N, const float* __restrict__ s,
                                                               const double* __restrict__ sorted,
                                                               const int* __restrict__ n_valid,
                                                               const RduState* __restrict__ state,
                                                               double* __restrict__ d) {
  __shared__ double v[kSortInit / 4];
  const RduState st = *state;
  const int m = *n_valid;
  const bool lds = m <= kSortInit / 4;  // block-uniform
  if (lds) {
    for (int j = threadIdx.x; j < m; j += kST) v[j] = sorted[j];
    __syncthreads();
  }
  auto nearest = [&](const double* q, double fi) {
    int lo = 0, hi = m;  // first index with q[idx] >= fi
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (q[mid] < fi) lo = mid + 1; else hi = mid;
    }
    double best = INFINITY;
    if (lo < m) best = fmin(best, fabs(fi - q[lo]));
    if (lo > 0) best = fmin(best, fabs(fi - q[lo - 1]));
    return best;
  };
  for (int i = blockIdx.x * kST + threadIdx.x; i < N; i += gridDim.x * kST) {
    if (s[i] != s[i] || m == 0) {
      d[i] = s[i] != s[i] ? -1.0 : INFINITY;
      continue;
    }
    const double fi = fhat(s, i, st);
    d[i] = lds ? nearest(v, fi) : nearest(sorted, fi);
  }
}

// d[i] = min over the initial labeled set of |f_i - f_j|
__global__ __launch_bounds__(kST) void rdu_dinit_kernel(int N, const float* __restrict__ s,
                                                        const int* __restrict__ init, int n_init,
                                                        const RduState* __restrict__ state,
                                                        double* __restrict__ d) {
  __shared__ double tf[kST];
  const RduState st = *state;
  const int i = blockIdx.x * kST + threadIdx.x;
  const double fi = i < N ? fhat(s, i, st) : 0.0;
  double best = INFINITY;
  for (int j0 = 0; j0 < n_init; j0 += kST) {
    __syncthreads();
    const int j = j0 + threadIdx.x;
    const int idx = j < n_init ? init[j] : -1;
    tf[threadIdx.x] = (idx >= 0 && idx < N) ? fhat(s, idx, st) : NAN;
    __syncthreads();
    const int n = min(kST, n_init - j0);
    for (int jj = 0; jj < n; ++jj) {
      const double fj = tf[jj];
      if (fj == fj) best = fmin(best, fabs(fi - fj));
    }
  }
  if (i < N) d[i] = s[i] == s[i] ? best : -1.0;  // an unscored (NaN) program is no candidate
}

// the initial labeled programs are not candidates
__global__ __launch_bounds__(kST) void rdu_mark_kernel(int N, const int* __restrict__ init, int n_init,
                                                       double* __restrict__ d) {
  const int j = blockIdx.x * kST + threadIdx.x;
  if (j < n_init) {
    const int i = init[j];
    if (i >= 0 && i < N) d[i] = -1.0;
  }
}

// One selection. Over the whole pool it reads every candidate's distance,
// type and prediction: 138 MB and 53 us for 8.65 M programs, 64 times. But from
// one selection to the next a candidate's t_s = f d + u can rise only by what
// u rises: d is a running minimum (Eq. (1)), and u (Eq. (2)-(3)) is one
// quadratic in f, whose largest change over f in [0, 1] is known in closed
// form. So a pass over the whole pool also collects the candidates with t_s >=
// cut, and the next launches run on that short list alone: while the list's
// best is at or above cut plus the rise since, no candidate outside it can
// win. When it no longer is, the launch selects nothing and the next one
// takes the whole pool again (at most `spare` times, so that n_select + spare
// launches always suffice). The cut comes from a histogram of a sample of t_s,
// for half the list's room; a list that overflows is not used.
// Scores that many candidates share, or that have a few far outliers, give
// lists that are empty, overflow or serve few selections. So lists are kept
// an account: the selections they served less `cost` for each try. When it is
// overdrawn, `wait` launches neither sample nor collect (kRduPlain, the pass
// that pools without the list get) before the next try, twice as many each time until a
// list serves more than its cost. The call over 140,000 / 1 M / 8.65 M programs,
// 64 selections, us: equal scores 1,605 / 2,713 / 4,425 without the account, 741 /
// 1,376 / 2,869 with it (722 / 1,908 / 3,545 with passes over the whole pool only,
// of 1,024 blocks); 64 different scores 1,306 / 2,913 / 3,789, 790 / 1,504 / 3,336
// (759 / 1,958 / 3,625).
// The arithmetic per candidate is the same in both, and ties go to the lower
// index, so the selection is too. The call over 8.65 M programs with 1,024
// initial ones, 64 selections: 3.6 ms with passes over the whole pool only,
// 1.10 to 1.20 ms now. Of that, in one traced call, five passes over the pool of 59 to 93
// us (the first samples; the others also collect, and fold in the up to 20 labels
// since the one before) take 392 us, 62 launches on lists of 6 to 9 us, bound by the
// latency of a chain of loads, block reductions and arrival, 507, the setup 115 and nine
// launches with nothing left to do 40.
constexpr int kRduUnroll = 4;
constexpr int kRduList = 32768;       // room of the short list
constexpr double kRiseMargin = 1e-12;  // far above the rounding of u_s and of its change (a few 1e-16)

constexpr int kRduPlainGrid = 512;     // blocks of a kRduPlain launch
constexpr int kRduMaxBalance = 256;    // selections that lists may be behind after a long good stretch

constexpr int kRduHeld = 256 + kST * kRduUnroll;  // of them held in LDS by a block: 256 and a round's

struct ListItem {
  double f, d;
  int i, op;
};

// block argmax of (t, i), lower index on ties, i < 0: none; every thread gets it
__device__ __forceinline__ Best block_best(double t, int i, double* st, int* si) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double t2 = __shfl_xor(t, o, 64);
    const int i2 = __shfl_xor(i, o, 64);
    if (i2 >= 0 && better(t2, i2, t, i)) {
      t = t2;
      i = i2;
    }
  }
  __syncthreads();  // st, si are free
  if ((threadIdx.x & 63) == 0) {
    st[threadIdx.x >> 6] = t;
    si[threadIdx.x >> 6] = i;
  }
  __syncthreads();
  t = st[0];
  i = si[0];
#pragma unroll
  for (int w = 1; w < kST / 64; ++w)
    if (si[w] >= 0 && better(st[w], si[w], t, i)) {
      t = st[w];
      i = si[w];
    }
  return Best{t, i};
}

__device__ __forceinline__ double rdu_t(double f, double d, const RduState& st, double inv) {
  const double mu = (f + st.S1) * inv;                 // Eq. (2)
  const double u = (f * f + st.S2) * inv - mu * mu;    // Eq. (3), from the running sums
  return f * d + u;
}

// The most that u_s rose, for any f in [0, 1], since the list was collected:
// the change is a f^2 + b f + c, largest at an end, or at the vertex when it
// opens downwards.
__device__ __forceinline__ double u_rise(const RduState& st) {
  const double v = 1.0 / (double)(st.M + 1), w = 1.0 / (double)(st.cut_M + 1);
  const double a = (v - v * v) - (w - w * w);
  const double b = -2.0 * (st.S1 * v * v - st.cut_S1 * w * w);
  const double c = (st.S2 * v - st.S1 * st.S1 * v * v) - (st.cut_S2 * w - st.cut_S1 * st.cut_S1 * w * w);
  double m = fmax(c, a + b + c);
  if (a < 0.0 && b > 0.0 && b < -2.0 * a) m = fmax(m, c - b * b / (4.0 * a));
  return m + kRiseMargin;
}

template <bool LIST>  // with the short list, else over the whole pool always
__global__ __launch_bounds__(kST) void rdu_score_kernel(int N, const float* __restrict__ s,
                                                        const int* __restrict__ op, int n_ops,
                                                        const double* __restrict__ budget,
                                                        int* __restrict__ sel, RduState* state,
                                                        double* __restrict__ d, Best* part, ListItem* list,
                                                        int* hist, int* out, int parity) {
  __shared__ double bt[kST / 64];
  __shared__ int bi[kST / 64];
  __shared__ double sfl[LIST ? kST : 1];
  __shared__ int sil[LIST ? kST : 1];
  __shared__ int sh[LIST ? kHistBins : 1];
  __shared__ ListItem held[LIST ? kRduHeld : 1];
  __shared__ int nheld, flag, above;
  const int tid = threadIdx.x, lane = tid & 63;
  const RduState st = *state;
  if (st.done) return;
  // A launch does not wait for the blocks that it has no work for (on the list,
  // and kRduPlain's past its grid), so one that starts late may find the next
  // launch's state here: its own launch's mode is kept, the last block writes
  // the other one.
  const int mode = LIST ? (parity ? st.mode[1] : st.mode[0]) : (int)kRduPlain;
  const double inv = 1.0 / (double)(st.M + 1);
  double best_t = 0.0;
  int best_i = -1;
  int blocks = gridDim.x;  // blocks that take part
  // one pass over the whole pool: FULL with every label since the last one
  // (the first kST of them from LDS), sampling and collecting; else with the
  // last label
  auto pool = [&](auto FULL) {
    constexpr bool kFull = decltype(FULL)::value;
    const int np = kFull ? st.count - st.ver : min(st.count, 1), npl = min(np, kST);
    const double last_f = !kFull && np ? fhat(s, st.last, st) : 0.0;
    if constexpr (kFull) {
      for (int b = tid; b < kHistBins; b += kST) sh[b] = 0;
      if (tid < npl) {
        sil[tid] = out[st.ver + tid];
        sfl[tid] = fhat(s, sil[tid], st);
      }
      if (tid == 0) nheld = 0;
      __syncthreads();
    }
    const double base = u_min(st.S1, st.S2, inv);
    const bool sampled = kFull && st.spare > 0 && st.wait == 0 && (blockIdx.x & (kHistEvery / 4 - 1)) == 0;
    bool collect = kFull && st.collect;  // block-uniform
    // the block's held items to the list, as far as it has room (the count
    // goes on, so an overfull list is noticed, and this block stops collecting)
    auto append = [&](int n) {
      if (tid == 0 && n) flag = atomicAdd(&state->nact, n);
      __syncthreads();
      for (int q = tid; q < n; q += kST)
        if (flag + q < kRduList) list[flag + q] = held[q];
      if (n && flag + n > kRduList) collect = false;
      __syncthreads();
      if (tid == 0) nheld = 0;
      __syncthreads();
    };
    constexpr int U = kRduUnroll;
    static_assert(U == 4, "the sample takes one of a round's four");
    for (int64_t j0 = (int64_t)blockIdx.x * kST * U; j0 < N; j0 += (int64_t)blocks * kST * U) {
      // every load at a clamped place and without a condition, so that a
      // round's twelve, then its eight lookups by type, are in flight together
      double dv[U], fv[U], bud[U];
      int iv[U], ov[U], sc[U];
      float sv[U];
      bool low[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        iv[k] = (int)min(j0 + k * kST + tid, (int64_t)N - 1);
        dv[k] = d[iv[k]];
        ov[k] = op[iv[k]];
        sv[k] = s[iv[k]];
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int o = min(max(ov[k], 0), n_ops - 1);
        sc[k] = sel[o];
        bud[k] = budget[o];
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        fv[k] = st.range > 0.0 ? ((double)sv[k] - st.lo) / st.range : 0.0;
        low[k] = false;
      }
      for (int p = 0; p < np; ++p) {
        const int il = !kFull ? st.last : p < npl ? sil[p] : out[st.ver + p];
        const double fl = !kFull ? last_f : p < npl ? sfl[p] : fhat(s, il, st);
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const double dn = il == iv[k] ? -1.0 : fabs(fv[k] - fl);  // a labeled program is no candidate
          if (dn < dv[k]) {
            dv[k] = dn;
            low[k] = true;
          }
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int i = iv[k], o = ov[k];
        if (dv[k] >= 0.0 && (o < 0 || o >= n_ops || (double)sc[k] >= bud[k])) {
          dv[k] = -1.0;  // its operator's budget is used up
          low[k] = true;
        }
        const bool in = j0 + k * kST + tid < N;
        if (in && low[k]) d[i] = dv[k];
        const bool cand = in && dv[k] >= 0.0;  // not labeled, masked or past the end
        const double t = cand ? rdu_t(fv[k], dv[k], st, inv) : 0.0;
        if (cand && better(t, i, best_t, best_i)) {
          best_t = t;
          best_i = i;
        }
        if constexpr (kFull) {
          // one atomic for the lanes that share the first one's bin, and one
          // for a wavefront's collected candidates: with equal scores 64 lanes
          // would queue at one address
          const uint64_t cands = __builtin_amdgcn_ballot_w64(cand);
          if (k == 0 && sampled && cands) {
            const int bin = cand ? hist_bin(t - base) : -1;
            const int first = __builtin_amdgcn_readlane(bin, __builtin_ctzll(cands));
            const uint64_t same = __builtin_amdgcn_ballot_w64(bin == first);
            if (bin == first) {
              if (lane == __builtin_ctzll(same)) atomicAdd(&sh[first], __builtin_popcountll(same));
            } else if (cand) {
              atomicAdd(&sh[bin], 1);
            }
          }
          const bool take = collect && cand && t >= st.cut;
          const uint64_t takes = __builtin_amdgcn_ballot_w64(take);
          if (takes) {
            const int first = __builtin_ctzll(takes);
            int at = 0;
            if (lane == first) at = atomicAdd(&nheld, __builtin_popcountll(takes));
            at = __builtin_amdgcn_readlane(at, first);
            if (take)
              held[at + __builtin_popcountll(takes & ((1ull << lane) - 1))] = ListItem{fv[k], dv[k], i, o};
          }
        }
      }
      if (kFull && collect) {
        __syncthreads();
        const int n = nheld;
        if (n > kRduHeld - kST * kRduUnroll) append(n);
        else __syncthreads();  // nheld is read before the next round adds to it
      }
    }
    if constexpr (kFull) {
      __syncthreads();
      if (collect) append(nheld);
      if (sampled)
        for (int b = tid; b < kHistBins; b += kST)
          if (sh[b]) atomicAdd(&hist[b], sh[b]);
    }
  };
  if (mode == kRduListed) {
    blocks = min((int)gridDim.x, max(1, (st.nact + kST - 1) / kST));
    if ((int)blockIdx.x >= blocks) return;
    for (int q = blockIdx.x * kST + tid; q < st.nact; q += blocks * kST) {
      ListItem it = list[q];
      const double dn = it.i == st.last ? -1.0 : fabs(it.f - fhat(s, st.last, st));
      if (it.d >= 0.0) {
        if ((double)sel[it.op] >= budget[it.op]) it.d = -1.0;
        else it.d = fmin(it.d, dn);
        list[q].d = it.d;
      }
      const double t = rdu_t(it.f, it.d, st, inv);
      if (it.d >= 0.0 && better(t, it.i, best_t, best_i)) {
        best_t = t;
        best_i = it.i;
      }
    }
  } else if (LIST && mode == kRduWhole) {
    if constexpr (LIST) pool(std::true_type{});
  } else {
    blocks = min((int)gridDim.x, kRduPlainGrid);
    if ((int)blockIdx.x >= blocks) return;
    pool(std::false_type{});
  }
  const Best b = block_best(best_t, best_i, bt, bi);
  if (tid == 0) {
    part[blockIdx.x] = b;
    __threadfence();  // the partial is visible before the arrival is counted
    flag = atomicAdd(&state->arrived, 1u) == (unsigned)blocks - 1;
  }
  __syncthreads();
  if (!flag) return;

  // the last block: every partial is in; reduce them and label the winner
  __threadfence();
  double t = 0.0;
  int i = -1;
  for (int q = tid; q < blocks; q += kST) {
    const Best pq = part[q];
    if (pq.i >= 0 && better(pq.t, pq.i, t, i)) {
      t = pq.t;
      i = pq.i;
    }
  }
  const Best w = block_best(t, i, bt, bi);
  int edge = kHistBins;
  const bool sampling = LIST && mode == kRduWhole && st.spare > 0 && st.wait == 0;
  if (sampling) {
    // the lowest bin edge that half the list's room would hold: a suffix sum
    // over the bins, lane l of one wavefront taking per bins from the top down
    for (int q = tid; q < kHistBins; q += kST) sh[q] = atomicExch(&hist[q], 0);
    if (tid == 0) {
      flag = kHistBins;
      above = 0;
    }
    __syncthreads();
    constexpr int per = (kHistBins + 63) / 64;
    int own[per], sum = 0, before = 0;
    if (tid < 64) {
#pragma unroll
      for (int r = 0; r < per; ++r) {
        const int q = kHistBins - 1 - (tid * per + r);
        sum += q >= 0 ? sh[q] : 0;
        own[r] = sum;
      }
      before = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(before, o, 64);
        if (tid >= o) before += v;
      }
      before -= sum;
#pragma unroll
      for (int r = 0; r < per; ++r) {
        const int q = kHistBins - 1 - (tid * per + r);
        if (q >= 0 && (before + own[r]) * (int64_t)kHistEvery <= kRduList / 2) atomicMin(&flag, q);
      }
    }
    __syncthreads();
    edge = flag;
    if (tid < 64) {
#pragma unroll
      for (int r = 0; r < per; ++r)
        if (kHistBins - 1 - (tid * per + r) == edge) above = before + own[r];
    }
    __syncthreads();
  }
  if (tid == 0) {
    state->arrived = 0;
    bool active = mode == kRduListed, collect = false;
    int spare = st.spare, balance = st.balance, wait = st.wait, next = kRduWhole;
    const int nact = LIST && st.collect ? atomicAdd(&state->nact, 0) : 0;  // as this launch left it
    double next_cut = st.next_cut;
    if (LIST && !active) state->ver = st.count;  // every label but this launch's is in the distances
    if (sampling) {
      state->next_cut = next_cut = u_min(st.S1, st.S2, inv) + hist_edge(min(edge, kHistBins - 1));
      collect = above > 0;  // no cut that a list could be collected with otherwise
    }
    // the list that this launch collected, if it is of use
    const bool listed = mode == kRduWhole && st.collect && nact >= 2 && nact <= kRduList;
    if (sampling && !listed && (!collect || st.collect)) balance -= st.cost;
    if (mode == kRduPlain && wait > 0) --wait;
    if (active && (w.i < 0 || !(w.t >= st.cut + u_rise(st)))) {
      // a candidate outside the list may be better: the whole pool next
      balance = min(balance + st.run - st.cost, kRduMaxBalance);
      if (st.run > st.cost) state->back = st.back0;
      --spare;
      active = false;
      collect = true;
    } else if (w.i < 0) {
      state->done = 1;
    } else {
      const double f = fhat(s, w.i, st);
      out[st.count] = w.i;
      state->count = st.count + 1;
      state->M = st.M + 1;
      state->S1 = st.S1 + f;
      state->S2 = st.S2 + f * f;
      state->last = w.i;
      sel[op[w.i]] += 1;
      if (st.count + 1 >= st.n_select) state->done = 1;
      state->run = st.run + 1;
      if (listed) {
        active = true;  // it holds every t_s >= cut
        state->cut_S1 = st.S1;
        state->cut_S2 = st.S2;
        state->cut_M = st.M;
        state->run = 0;
      }
    }
    if constexpr (LIST) {
      if (balance < 0) {
        balance = 0;
        wait = st.back;
        state->back = min(2 * st.back, 1 << 20);
      }
      // distances without the labels of a list's run need kRduWhole
      if (mode != kRduListed && (wait > 0 || spare == 0)) next = kRduPlain;
      collect = collect && !active && next == kRduWhole && wait == 0 && spare > 0;
      state->mode[parity ^ 1] = active ? (int)kRduListed : next;
      state->spare = spare;
      state->balance = balance;
      state->wait = wait;
      if (!active) state->nact = 0;
      state->collect = collect;
      if (collect) state->cut = next_cut;
    }
  }
}

__global__ __launch_bounds__(kST) void rdu_finish_kernel(int n_select, const RduState* __restrict__ state,
                                                         int* __restrict__ out, int* __restrict__ count) {
  const int c = state->count;
  for (int i = threadIdx.x; i < n_select; i += kST)
    if (i >= c) out[i] = -1;
  if (threadIdx.x == 0) *count = c;
}

constexpr int kRduGrid = 1024;  // blocks of the grid passes (grid-stride)

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// ---------------------------------------------------------------- Top-k score (Eq. (12))
// One workgroup per segment: the lowest latency of the segment and the
// lowest among its k best-ranked candidates (indices from topk_kernel), each
// times the segment's weight. fp32 latencies and weights multiply exactly in
// fp64. An empty segment contributes (0, 0).
__global__ __launch_bounds__(kST) void topk_score_seg_kernel(const int* __restrict__ offs, int k,
                                                             const int* __restrict__ top,
                                                             const float* __restrict__ lat,
                                                             const float* __restrict__ w,
                                                             double* __restrict__ part) {
  __shared__ float sA[kST / 64], sB[kST / 64];
  const int g = blockIdx.x, tid = threadIdx.x;
  const int lo = offs[g], hi = offs[g + 1];
  float mAll = __builtin_inff(), mTop = __builtin_inff();
  for (int i = lo + tid; i < hi; i += kST) mAll = fminf(mAll, lat[i]);
  for (int j = tid; j < k; j += kST) {
    const int i = top[(int64_t)g * k + j];
    if (i >= 0) mTop = fminf(mTop, lat[i]);
  }
  for (int o = 32; o > 0; o >>= 1) {
    mAll = fminf(mAll, __shfl_xor(mAll, o));
    mTop = fminf(mTop, __shfl_xor(mTop, o));
  }
  if ((tid & 63) == 0) {
    sA[tid >> 6] = mAll;
    sB[tid >> 6] = mTop;
  }
  __syncthreads();
  if (tid == 0) {
    float a = sA[0], b = sB[0];
    for (int v = 1; v < kST / 64; ++v) {
      a = fminf(a, sA[v]);
      b = fminf(b, sB[v]);
    }
    const bool empty = hi <= lo;
    part[2 * g] = empty ? 0.0 : (double)w[g] * (double)a;
    part[2 * g + 1] = empty ? 0.0 : (double)w[g] * (double)b;
  }
}

// One workgroup: both sums over the segments in a fixed order (a strided
// serial pass per thread, then a fixed tree), so the result is deterministic.
__global__ __launch_bounds__(1024) void topk_score_sum_kernel(int n_seg, const double* __restrict__ part,
                                                              double* __restrict__ out) {
  __shared__ double sN[1024], sD[1024];
  const int tid = threadIdx.x;
  double n = 0.0, d = 0.0;
  for (int g = tid; g < n_seg; g += 1024) {
    n += part[2 * g];
    d += part[2 * g + 1];
  }
  sN[tid] = n;
  sD[tid] = d;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (tid < o) {
      sN[tid] += sN[tid + o];
      sD[tid] += sD[tid + o];
    }
    __syncthreads();
  }
  if (tid == 0) {
    out[0] = sN[0] / sD[0];
    out[1] = sN[0];
    out[2] = sD[0];
  }
}

}  // namespace

size_t topk_score_workspace_bytes(int n_seg, int k) {
  return al256((size_t)n_seg * k * 4) + al256((size_t)n_seg * 2 * 8);
}

hipError_t launch_topk_score(int n_seg, const int* offs, const float* s, const float* lat, const float* w,
                             int k, double* out, void* ws, hipStream_t st) {
  if (n_seg <= 0 || k < 1 || k > 1024) return hipErrorInvalidValue;
  int* top = static_cast<int*>(ws);
  double* part = reinterpret_cast<double*>(static_cast<char*>(ws) + al256((size_t)n_seg * k * 4));
  hipError_t e = launch_topk(n_seg, offs, s, k, top, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(topk_score_seg_kernel, dim3(n_seg), dim3(kST), 0, st, offs, k, top, lat, w, part);
  hipLaunchKernelGGL(topk_score_sum_kernel, dim3(1), dim3(1024), 0, st, n_seg, part, out);
  return hipGetLastError();
}

hipError_t launch_topk(int n_seg, const int* offs, const float* s, int K, int* out, hipStream_t st) {
  if (n_seg <= 0 || K < 1 || K > 1024) return hipErrorInvalidValue;
#define TCL_TOPK(PP) hipLaunchKernelGGL((topk_kernel<PP>), dim3(n_seg), dim3(kTK), 0, st, offs, s, K, out)
  if (K <= 64) TCL_TOPK(256);
  else if (K <= 256) TCL_TOPK(512);
  else TCL_TOPK(1536);
#undef TCL_TOPK
  return hipGetLastError();
}

size_t rdu_workspace_least_bytes(int N, int n_ops) {
  const int grid = std::min((N + kST - 1) / kST, kRduGrid);
  return al256(sizeof(RduState)) + al256((size_t)N * 8) + al256((size_t)n_ops * 8) +
         al256((size_t)(n_ops + 1) * 4) * 2 + al256((size_t)grid * 2 * 4) + al256((size_t)grid * sizeof(Best)) +
         al256((size_t)kSortInit * 8) + 256;
}

// the short list and its histogram, for pools that may use them
constexpr int kRduListMinN = 4 * kRduList + 1;
size_t rdu_workspace_bytes(int N, int n_ops) {
  return rdu_workspace_least_bytes(N, n_ops) +
         (N >= kRduListMinN ? al256((size_t)kRduList * sizeof(ListItem)) + al256((size_t)kHistBins * 4) : 0);
}

hipError_t launch_rdu_select(int N, const float* s, const int* op, int n_ops, const int* init, int n_init,
                             int n_select, int* out, int* count, void* ws, size_t ws_bytes, hipStream_t st) {
  if (N <= 0 || n_ops <= 0 || n_ops > kMaxOps || n_init < 0 || n_select < 0) return hipErrorInvalidValue;
  if (ws_bytes < rdu_workspace_least_bytes(N, n_ops)) return hipErrorInvalidValue;
  const int grid = std::min((N + kST - 1) / kST, kRduGrid);
  char* p = static_cast<char*>(ws);
  RduState* state = reinterpret_cast<RduState*>(p);
  p += al256(sizeof(RduState));
  double* d = reinterpret_cast<double*>(p);
  p += al256((size_t)N * 8);
  double* budget = reinterpret_cast<double*>(p);
  p += al256((size_t)n_ops * 8);
  int* opcount = reinterpret_cast<int*>(p);
  p += al256((size_t)(n_ops + 1) * 4);
  int* sel = reinterpret_cast<int*>(p);
  p += al256((size_t)(n_ops + 1) * 4);
  float* mm = reinterpret_cast<float*>(p);
  p += al256((size_t)grid * 2 * 4);
  Best* part = reinterpret_cast<Best*>(p);
  p += al256((size_t)grid * sizeof(Best));
  double* sorted = reinterpret_cast<double*>(p);
  p += al256((size_t)kSortInit * 8);
  int* n_valid = reinterpret_cast<int*>(p);
  p += 256;

  hipLaunchKernelGGL(rdu_zero_kernel, dim3(std::max(1, std::min((n_ops + kST) / kST, 64))), dim3(kST), 0, st,
                     n_ops + 1, opcount);
  hipLaunchKernelGGL(rdu_stats_kernel, dim3(grid), dim3(kST), 0, st, N, s, op, n_ops, mm, opcount);
  // The short list pays where passes over the whole pool are long and the
  // labeled set is dense enough in the pool for few candidates to be near the
  // best t_s. Measured, us per selection with the list / without: 8.65 M
  // programs with 1,024, 256, 128 and 64 initial ones 17 / 57, 40 / 57, 61 / 57
  // and 63 / 57, 1 M with 64 and 32 13.6 / 28 and 24 / 28, 262,000 with 32 10.9 /
  // 13.1, 100,000 with 64 9.6 / 9.6, 40,000 with 64 9.3 / 8.5.
  // A workspace without room for it is served as it always was, by plain passes.
  const bool use_list = N >= kRduListMinN && n_init >= 32 && (int64_t)n_init * 40000 >= N &&
                        ws_bytes >= rdu_workspace_bytes(N, n_ops);
  ListItem* list = nullptr;
  int* hist = nullptr;
  if (use_list) {
    list = reinterpret_cast<ListItem*>(p);
    p += al256((size_t)kRduList * sizeof(ListItem));
    hist = reinterpret_cast<int*>(p);
  }
  // launches beyond n_select that may select nothing
  const int spare = use_list ? n_select / 8 + 4 : 0;
  hipLaunchKernelGGL(rdu_setup_kernel, dim3(1), dim3(kST), 0, st, N, s, n_ops, init, n_init, n_select, mm, grid,
                     opcount, budget, sel, spare, hist, state);
  if (n_init <= kSortInit) {
    hipLaunchKernelGGL(rdu_sort_init_kernel, dim3(1), dim3(1024), 0, st, N, s, init, n_init, state, sorted, n_valid);
    hipLaunchKernelGGL(rdu_dinit_sorted_kernel, dim3(grid), dim3(kST), 0, st, N, s, sorted, n_valid, state, d);
  } else {
    hipLaunchKernelGGL(rdu_dinit_kernel, dim3((N + kST - 1) / kST), dim3(kST), 0, st, N, s, init, n_init, state, d);
  }
  if (n_init > 0)
    hipLaunchKernelGGL(rdu_mark_kernel, dim3((n_init + kST - 1) / kST), dim3(kST), 0, st, N, init, n_init, d);
  // a block's arrival costs more than a longer loop: 8.65 M programs 50.6 us a
  // pass with 512 blocks, 53.0 with 768, 57.1 with 1,024; 1 M 19.6, 24.5, 28.3.
  // With the list, whose few passes collect too: 1.19 ms a call with 512, 1.10
  // with 1,024
  const int sgrid = (int)std::min<int64_t>(((int64_t)N + kST * kRduUnroll - 1) / (kST * kRduUnroll),
                                           use_list ? kRduGrid : kRduPlainGrid);
  for (int it = 0; it < n_select + spare; ++it)
    hipLaunchKernelGGL(use_list ? rdu_score_kernel<true> : rdu_score_kernel<false>, dim3(sgrid), dim3(kST), 0, st, N, s,
                       op, n_ops, budget, sel, state, d, part, list, hist, out, it & 1);
  hipLaunchKernelGGL(rdu_finish_kernel, dim3(1), dim3(kST), 0, st, n_select, state, out, count);
  return hipGetLastError();
}

}  // namespace tcl
