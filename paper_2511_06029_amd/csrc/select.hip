// Retention masks by radix selection, gfx950.
//
// Three rules share one kernel template:
//  * RASR per segment: one block per (layer, sequence, KV head); the rank key
//    is that head's accumulated score.
//  * RASR shared by the heads of a layer: one block per (layer, sequence); the
//    key is the head-summed score (Eq. 2 collapses attention over heads), the
//    fp32 sum in ascending head order, and the mask goes to every head.
//  * Algorithm 1 (segmented token shrinking) with the size trigger: one block
//    per (layer, sequence) on the head-summed score.  The breakpoint needs no
//    sort: the head-to-cut ratio test holds on a suffix of the ranking (the
//    values never increase along it), so one max pass and one counting pass
//    give the first rank where it holds, and the breakpoint is the first cut
//    point at or after it.  The salient set is then the top-`breakpoint`
//    selection below.
//
// Selection: fp32 keys map to 32-bit words whose unsigned order is the float
// order (+0 and -0 equal, NaN below every number).  An MSB-first radix select
// with 8-bit digits and a 256-bin LDS histogram finds the exact key T of the
// m-th best candidate, how many candidates equal to T are still needed and
// how many there are.  When all of them are needed (the usual case) one
// elementwise pass keeps the candidates at or above T; otherwise an ordered
// pass keeps every candidate above T and the lowest-indexed ones equal to T.
// Candidate sets of up to kRegKeys rows per thread are read once into
// registers, and the radix passes and the elementwise pass use those; larger
// sets are re-read per pass, each thread issuing the loads of eight rows
// before it uses the first.
#include "device_common.h"
#include "lethe_internal.h"

namespace lethe {

namespace {

__device__ inline uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;  // NaN ranks last
  if (u == 0x80000000u) u = 0u;                      // -0 ties with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inverse of order_key on the keys of numbers (NaN's key 0 is never inverted).
__device__ inline float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Rank value of row j: one head's score, or the fp32 head sum (additions in
// ascending head order, each rounded; no multiply, so nothing contracts).
template <bool kShared, int W>
struct Scores {
  const float* s;       // head 0's segment
  long long hstride;    // rows between the segments of consecutive heads
  int heads;
  __device__ inline float operator()(int j) const {
    if constexpr (!kShared) {
      return s[j];
    } else {
      float acc = s[j];
      for (int h = 1; h < heads; ++h) acc = acc + s[h * hstride + j];
      return acc;
    }
  }
  // The same for rows j[0 .. U) (valid indices): the loads of the U rows and
  // of W heads are issued together, unconditionally (a head at a time they
  // cost one memory latency each; a last group short of W heads reads its last
  // one again).
  template <int U>
  __device__ inline void batch(const int* j, float* v) const {
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = s[j[u]];
    if constexpr (kShared) {
      for (int h0 = 1; h0 < heads; h0 += W) {
        float x[W][U];
#pragma unroll
        for (int hh = 0; hh < W; ++hh)
#pragma unroll
          for (int u = 0; u < U; ++u) x[hh][u] = s[min(h0 + hh, heads - 1) * hstride + j[u]];
#pragma unroll
        for (int hh = 0; hh < W; ++hh)
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (h0 + hh < heads) v[u] = v[u] + x[hh][u];
      }
    }
  }
};

template <int NT>
struct SelectShared {
  uint32_t hist[2][256];
  uint32_t digit, need, count;
  uint32_t red_u[NT / kWave];
  uint32_t red_c[NT / kWave];
  long long scan_tmp[NT / kWave + 1];
  int plan[4];  // lo, hi, m, keep-all flag
};

// Rows a thread loads before it uses the first of them (the passes are bound
// by load latency).
constexpr int kU = 8;

// MSB-first radix select over candidates that `count_digits(hist, shift,
// prefix, pmask)` counts by the 8-bit digit at `shift` (those whose bits under
// pmask equal prefix): key T of the m-th best (m >= 1), how many candidates
// with key T belong to the best m, and how many have it; all threads get the
// three.  A digit whose candidates are all needed ends the search: T is then
// the lowest key of that digit, and the two counts are equal.  With keys that
// spread (accumulated attention) two or three of the four passes run.
// Bound by latency: two barriers a pass, the next histogram cleared while the
// first wave searches this one (five barriers and always four passes took 91 us
// for the 32768 segments of a batch-128 round, 1024 to 65536 rows at shares of
// 2% to 20%; this, 79 us).
template <int NT, class CountFn>
__device__ void radix_select(const CountFn& count_digits, uint32_t m, SelectShared<NT>& sh, uint32_t* T_out,
                             uint32_t* need_out, uint32_t* count_out) {
  const int tid = threadIdx.x;
  uint32_t prefix = 0, pmask = 0, need = m, count = 0;
  if (tid < 256) sh.hist[0][tid] = 0;
  __syncthreads();
  int cur = 0;
  for (int shift = 24; shift >= 0; shift -= 8, cur ^= 1) {
    count_digits(sh.hist[cur], shift, prefix, pmask);
    __syncthreads();
    if (tid < kWave) {
      // suffix[d] = matching keys whose digit is >= d: four bins a lane; the
      // digit is the largest one whose suffix reaches need.
      const uint32_t h0 = sh.hist[cur][4 * tid], h1 = sh.hist[cur][4 * tid + 1];
      const uint32_t h2 = sh.hist[cur][4 * tid + 2], h3 = sh.hist[cur][4 * tid + 3];
      const uint32_t tot = h0 + h1 + h2 + h3;
      uint32_t incl = tot;  // sum over lanes tid .. 63
      for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t v = __shfl_down(incl, o);
        if (tid + o < kWave) incl += v;
      }
      const uint32_t s4 = incl - tot, s3 = s4 + h3, s2 = s3 + h2, s1 = s2 + h1;
      if (incl >= need && s4 < need) {
        const int d = s3 >= need ? 3 : s2 >= need ? 2 : s1 >= need ? 1 : 0;
        sh.digit = (uint32_t)(4 * tid + d);
        sh.need = need - (d == 3 ? s4 : d == 2 ? s3 : d == 1 ? s2 : s1);
        sh.count = d == 3 ? h3 : d == 2 ? h2 : d == 1 ? h1 : h0;
      }
    }
    // The other histogram, for the next pass (by the last threads: the first
    // wave is busy).
    if (tid >= NT - 256) sh.hist[cur ^ 1][tid - (NT - 256)] = 0;
    __syncthreads();
    prefix |= sh.digit << shift;
    pmask |= 255u << shift;
    need = sh.need;
    count = sh.count;
    if (need == count) break;
  }
  *T_out = prefix;
  *need_out = need;
  *count_out = count;
}

// Keys a thread keeps in registers: candidate sets of up to kRegKeys * NT rows
// are read from memory once.
constexpr int kRegKeys = 32;

// Block-wide max of a key and sum of a count; every thread gets both.
template <int NT>
__device__ void block_max_count(uint32_t key, uint32_t cnt, SelectShared<NT>& sh, uint32_t* kmax,
                                uint32_t* csum) {
  for (int o = kWave / 2; o > 0; o >>= 1) {
    key = max(key, (uint32_t)__shfl_xor(key, o));
    cnt += (uint32_t)__shfl_xor(cnt, o);
  }
  const int w = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) {
    sh.red_u[w] = key;
    sh.red_c[w] = cnt;
  }
  __syncthreads();
  uint32_t k = 0, c = 0;
  for (int i = 0; i < NT / kWave; ++i) {
    k = max(k, sh.red_u[i]);
    c += sh.red_c[i];
  }
  __syncthreads();
  *kmax = k;
  *csum = c;
}

template <int NT, int MODE, int W>
__global__ __launch_bounds__(NT) void select_kernel(SelectArgs a) {
  constexpr bool kShared = MODE != kSelectRasr;
  constexpr bool kShrink = MODE == kSelectShrink;
  const int h = kShared ? 0 : (int)(blockIdx.x % a.HK);
  const int lb = kShared ? (int)blockIdx.x : (int)(blockIdx.x / a.HK);
  const int b = lb % a.B;
  const int l = lb / a.B;
  const int tid = threadIdx.x;
  const int n = a.len[(long long)l * a.B + b];
  const int c = a.cap[b];
  const long long base = a.seq_base[b];
  if (n < 0 || c < 0 || n > c || base < 0 || base + (long long)a.HK * c > a.rows_per_layer) {
    if (tid == 0) atomicOr(a.dev_status, LETHE_DEV_BAD_LAYOUT);
    return;
  }
  const long long row0 = (long long)l * a.rows_per_layer + base + (long long)h * c;
  const Scores<kShared, W> rank{a.score + row0, (long long)c, a.HK};
  uint8_t* keep = a.keep + row0;
  const int nheads = kShared ? a.HK : 1;
  __shared__ SelectShared<NT> sh;

  // The keys of rows [from, to) in registers, read once (eight rows' loads at
  // a time, two where the head sums of two rows a thread are all): row from +
  // u NT + tid is slot u.  Every pass over them leaves out the groups of eight
  // slots past the last row by a block-uniform branch, and no slot's liveness
  // is kept: as 32 stored lane masks it spilled scalar registers (154 of
  // them in Algorithm 1's kernel), and passes over 32 slots whatever the length
  // took 64.2 us for Algorithm 1 on 1024 lists of 1000 rows and two heads and
  // 40.2 us for the per-head masks of 8192 segments of 1000 rows (as it is, 38.8
  // and 27.6 us).
  uint32_t key[kRegKeys];
  auto load_keys = [&](int from, int to) {
    if (kShared && to - from <= 2 * NT) {
      int jj[2];
      float v[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) jj[u] = min(from + u * NT + tid, to - 1);
      rank.template batch<2>(jj, v);
#pragma unroll
      for (int u = 0; u < 2; ++u) key[u] = order_key(v[u]);
      return;
    }
#pragma unroll
    for (int u0 = 0; u0 < kRegKeys; u0 += kU) {
      if (from + u0 * NT < to) {
        int jj[kU];
        float v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) jj[u] = min(from + (u0 + u) * NT + tid, to - 1);
        rank.template batch<kU>(jj, v);
#pragma unroll
        for (int u = 0; u < kU; ++u) key[u0 + u] = order_key(v[u]);
      }
    }
  };
  // fn(key, row) for this thread's keys.
  auto each_key = [&](int from, int to, const auto& fn) {
#pragma unroll
    for (int u0 = 0; u0 < kRegKeys; u0 += kU) {
      if (from + u0 * NT < to) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int j = from + (u0 + u) * NT + tid;
          if (j < to) fn(key[u0 + u], j);
        }
      }
    }
  };

  // Plan: candidate rows [lo, hi), how many of them to keep (m), and the
  // forced rows, which are [0, fs) and [fr, n).
  int lo = 0, hi = 0, m = 0, fs = 0, fr = n;
  bool all = false;
  if constexpr (!kShrink) {
    int k = a.budget[(long long)b * a.L + l];
    if (k < 0) k = 0;
    if (k >= n) {
      all = true;
    } else {
      const int r = min(a.recent, k);
      const int sk = min(a.sink, k - r);
      m = k - r - sk;
      lo = sk;
      hi = n - r;
      fs = sk;
      fr = n - r;
    }
  } else {
    const long long lev0 = max(a.evict[(long long)l * a.B + b], 0);
    long long lev = lev0;
    long long bp = kShrinkNotTriggered;
    if (n <= lev0) {
      all = true;
    } else {
      // Head of the ranking and the NaN count (whose key is 0, and only
      // theirs), from registers where they hold every row (three passes over
      // memory and the radix passes: 42 us for 256 lists of 3000 to 6200 rows
      // and 8 heads; one pass: 27 us).
      const bool regs = n <= kRegKeys * NT;
      uint32_t kmax = 0, nnan = 0;
      {
        uint32_t km = 0, cn = 0;
        if (regs) {
          load_keys(0, n);
          each_key(0, n, [&](uint32_t k, int) {
            km = max(km, k);
            cn += k == 0u ? 1u : 0u;
          });
        } else {
          for (int j = tid; j < n; j += NT) {
            const float v = rank(j);
            km = max(km, order_key(v));
            cn += (v != v) ? 1u : 0u;
          }
        }
        block_max_count<NT>(km, cn, sh, &kmax, &nnan);
      }
      bp = kShrinkNoBreakpoint;
      const float head = key_value(kmax);
      if (kmax != 0u && head > 0.0f && a.segments > 1) {
        // cnt = rows whose ratio head / value stays below tau (tau * value >
        // head, exact in fp64): ranks [cnt, n - nnan) pass the test.
        const double dh = (double)head, dt = (double)a.tau;
        uint32_t cn = 0, unused = 0;
        if (regs) {
          each_key(0, n, [&](uint32_t k, int) { cn += (k != 0u && dt * (double)key_value(k) > dh) ? 1u : 0u; });
        } else {
          for (int j = tid; j < n; j += NT) {
            const float v = rank(j);
            cn += (v == v && dt * (double)v > dh) ? 1u : 0u;
          }
        }
        uint32_t cnt = 0;
        block_max_count<NT>(0u, cn, sh, &unused, &cnt);
        const long long D = a.segments;
        long long d = ((long long)cnt * D + n - 1) / n;  // first d with n*d >= cnt*D
        if (d < 1) d = 1;
        if (d <= D - 1) {
          const long long cut = ((long long)n * d) / D;
          if (cut < (long long)n - (long long)nnan) bp = cut;
        }
      }
      if (bp >= 0) {
        m = (int)bp;
        lo = 0;
        hi = n;
        fs = min(a.sink, n);
        fr = n - min(a.recent, n);
        lev = max(lev0, bp + (long long)a.recent);
      } else {
        all = true;
        lev = 2 * lev0;
      }
      if (lev > 0x7fffffffLL) lev = 0x7fffffffLL;
    }
    if (tid == 0) {
      a.evict[(long long)l * a.B + b] = (int32_t)lev;
      if (a.breakpoint) a.breakpoint[(long long)l * a.B + b] = (int32_t)bp;
    }
  }

  if (all) {
    for (int hh = 0; hh < nheads; ++hh)
      for (int j = tid; j < n; j += NT) keep[(long long)hh * c + j] = 1;
    return;
  }
  uint32_t T = 0, need = 0, countT = 0;
  if (m > 0 && hi - lo <= kRegKeys * NT) {
    if constexpr (!kShrink) load_keys(lo, hi);
    auto count_digits = [&](uint32_t* hist, int shift, uint32_t prefix, uint32_t pmask) {
      each_key(lo, hi, [&](uint32_t k, int) {
        if ((k & pmask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
      });
    };
    radix_select<NT>(count_digits, (uint32_t)m, sh, &T, &need, &countT);
    if (need == countT) {
      // Forced rows, then every candidate at or above T.
      for (int j = tid; j < fs; j += NT)
        for (int hh = 0; hh < nheads; ++hh) keep[(long long)hh * c + j] = 1;
      for (int j = max(fr, hi) + tid; j < n; j += NT)
        for (int hh = 0; hh < nheads; ++hh) keep[(long long)hh * c + j] = 1;
      each_key(lo, hi, [&](uint32_t k, int j) {
        const uint8_t kp = (j < fs || j >= fr || k >= T) ? 1 : 0;
        for (int hh = 0; hh < nheads; ++hh) keep[(long long)hh * c + j] = kp;
      });
      return;
    }
  } else if (m > 0) {
    auto count_digits = [&](uint32_t* hist, int shift, uint32_t prefix, uint32_t pmask) {
      for (int j0 = lo; j0 < hi; j0 += kU * NT) {
        int jj[kU];
        float v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) jj[u] = min(j0 + u * NT + tid, hi - 1);
        rank.template batch<kU>(jj, v);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const uint32_t k = order_key(v[u]);
          if (j0 + u * NT + tid < hi && (k & pmask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
        }
      }
    };
    radix_select<NT>(count_digits, (uint32_t)m, sh, &T, &need, &countT);
  }
  if (m == 0 || need == countT) {
    // Every candidate with key T is kept (or none is a candidate to keep):
    // no tie to break, so each row is decided on its own.
    for (int j0 = 0; j0 < n; j0 += kU * NT) {
      float v[kU];
      if (m > 0) {
        int jj[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) jj[u] = min(max(j0 + u * NT + tid, lo), hi - 1);
        rank.template batch<kU>(jj, v);
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int j = j0 + u * NT + tid;
        if (j < n) {
          const bool cand = m > 0 && j >= lo && j < hi;
          const uint8_t kp = (j < fs || j >= fr || (cand && order_key(v[u]) >= T)) ? 1 : 0;
          for (int hh = 0; hh < nheads; ++hh) keep[(long long)hh * c + j] = kp;
        }
      }
    }
    return;
  }
  // Ordered pass: ties with key T are taken by increasing row index.
  long long carry = 0;
  for (int j0 = 0; j0 < n; j0 += NT) {
    const int j = j0 + tid;
    const bool cand = j >= lo && j < hi && j < n;
    const uint32_t key = (cand && m > 0) ? order_key(rank(j)) : 0u;
    const bool eq = cand && m > 0 && key == T;
    long long total;
    const long long pos = block_excl_scan<NT>(eq ? 1 : 0, sh.scan_tmp, &total);
    if (j < n) {
      const bool forced = j < fs || j >= fr;
      const bool chosen = cand && m > 0 && (key > T || (eq && carry + pos < (long long)need));
      const uint8_t kp = (forced || chosen) ? 1 : 0;
      for (int hh = 0; hh < nheads; ++hh) keep[(long long)hh * c + j] = kp;
    }
    carry += total;
  }
}

// The heads after the first in as few groups of up to four as hold them, evenly
// cut.  Groups of four whatever the number read heads twice: 32 lists of 50000
// rows (read in every pass) took 82.9, 87.4 and 141.7 us with two, three and six
// heads, 71.3, 81.6 and 134.1 with a head at a time, and take 70.2, 74.8 and
// 129.5 this way.
template <int MODE>
lethe_status launch_head_sum(const SelectArgs& a, unsigned nb, hipStream_t s) {
  const int groups = (a.HK - 1 + 3) / 4;
  const int w = groups > 0 ? (a.HK - 1 + groups - 1) / groups : 1;
  const auto kernel = w == 1   ? select_kernel<1024, MODE, 1>
                      : w == 2 ? select_kernel<1024, MODE, 2>
                      : w == 3 ? select_kernel<1024, MODE, 3>
                               : select_kernel<1024, MODE, 4>;
  hipLaunchKernelGGL(kernel, dim3(nb), dim3(1024), 0, s, a);
  return hipGetLastError() == hipSuccess ? LETHE_OK : LETHE_ERR_HIP;
}

}  // namespace

lethe_status launch_select(const SelectArgs& a, hipStream_t s) {
  const long long nb = (long long)a.L * a.B * (a.mode == kSelectRasr ? a.HK : 1);
  if (nb > 0x7fffffffLL) return LETHE_ERR_UNSUPPORTED;
  if (nb == 0) return LETHE_OK;
  switch (a.mode) {
    case kSelectRasr:
      hipLaunchKernelGGL((select_kernel<256, kSelectRasr, 1>), dim3((unsigned)nb), dim3(256), 0, s, a);
      return hipGetLastError() == hipSuccess ? LETHE_OK : LETHE_ERR_HIP;
    case kSelectRasrShared:
      return launch_head_sum<kSelectRasrShared>(a, (unsigned)nb, s);
    case kSelectShrink:
      return launch_head_sum<kSelectShrink>(a, (unsigned)nb, s);
  }
  return LETHE_ERR_INVALID;
}

}  // namespace lethe
