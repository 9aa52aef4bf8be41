// Causal prefill attention that seeds the importance scores (Eq. 2 summed
// over the prompt's queries and the query heads of each KV group), gfx950.
//
// The qlen newest rows of each (sequence, KV head) segment come with queries;
// query i sits at position p = n - qlen + i and attends rows 0 .. p.  Two
// launches, both on v_mfma_f32_32x32x16_bf16:
//
//  1. prefill_fwd_kernel: flash attention forward.  A wavefront's unit is 32
//     query positions of one head; a block holds four consecutive units of a
//     KV group (ordered by position, then head) and walks the keys in 64-row
//     steps, K and V tiles shared by the waves through LDS (direct loads,
//     double buffered).  S^T = K Q^T, online softmax in base 2 with one query
//     per lane column, O^T = V^T P^T with P split into bf16 high and low
//     parts for fp32-level accuracy.  Writes out and each query's final
//     (max, 1 / sum).
//  2. prefill_score_kernel: key-major.  A wavefront keeps its keys in
//     registers and walks every later query tile of every head of the group,
//     recomputing S^T and summing exp2(x - max) / sum over the queries.
//     The query tiles go round robin to the block's item groups, whose sums
//     are added in order, and each key's total is added to its score once, so
//     there are no atomics and the result does not depend on scheduling.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "lethe_internal.h"

namespace lethe {

namespace {

constexpr int kPfThreads = 256;
constexpr int kPfWaves = kPfThreads / kWave;
constexpr float kPfNegBig = -1.0e30f;
constexpr long long kPfResident = 512;  // forward blocks the chip holds at once

typedef __bf16 pf_bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 pf_bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 pf_bf16x2_t __attribute__((ext_vector_type(2)));
typedef float pf_f32x2_t __attribute__((ext_vector_type(2)));
typedef float pf_f32x16_t __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) pf_bf16x4_t pf_lds_bf16x4_t;
typedef __attribute__((address_space(3))) char pf_lds_char_t;
typedef __attribute__((address_space(3))) void pf_lds_void_t;
typedef __attribute__((address_space(1))) const void pf_global_cvoid_t;

template <int D>
struct PfCfg {
  static constexpr int KS = D / 16;          // k-steps of 16 over the head dim
  static constexpr int NT = D / 32;          // output tiles of 32 dims
  static constexpr int ROWB = D * 2;         // bytes per bf16 row
  static constexpr int CH = ROWB / 16;       // 16-byte chunks per row
  static constexpr int STEP = 64;            // key rows per step
  // K / Q tiles: chunk c of row r at 16-byte slot r CH + (c ^ (r mod CH)), so
  // the 16 rows an operand read touches fall in different LDS banks.
  static constexpr int KTILE = STEP * ROWB;
  static constexpr int KLOADS = KTILE / (kWave * 16);
  static __device__ constexpr int kslot(int r, int c) { return r * CH + (c ^ (r % CH)); }
  // V tiles: load u (one wavefront, 16 bytes a lane) carries rows
  // u + VLOADS j into block u; the blocks' padding spreads the rows of one
  // transposing read over the LDS banks.
  static constexpr int LPR = ROWB / 16;
  static constexpr int RPL = kWave / LPR;
  static constexpr int VLOADS = STEP / RPL;
  static constexpr int VBLK = kWave * 16 + 64;
  static constexpr int VTILE = VLOADS * VBLK;
  static __device__ constexpr int vaddr(int r, int c) { return (r % VLOADS) * VBLK + (r / VLOADS) * ROWB + c; }
};

// Waits for every vector-memory load (expcnt and lgkmcnt left free).
__device__ inline void wait_vmem() { __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8)); }

__device__ inline pf_bf16x8_t pf_zero8() {
  pf_bf16x8_t z;
#pragma unroll
  for (int j = 0; j < 8; ++j) z[j] = (__bf16)0.0f;
  return z;
}

// 16 bytes a lane from `base + off` (base wave-uniform) into LDS: lane l's
// land at dst + 16 l.
__device__ inline void pf_load_lds(const char* base, unsigned off, pf_lds_char_t* dst) {
  __builtin_amdgcn_global_load_lds((pf_global_cvoid_t*)(base + off), (pf_lds_void_t*)dst, 16, 0, 0);
}

// The larger of v and the other 32-lane half's.
__device__ inline float pf_max_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Sizes of one sequence, or false (flagged) when they do not fit together.
struct PfSeq {
  int n, qlen, first;
  long long q0, row0;
};

__device__ inline bool pf_seq(const PrefillArgs& a, int b, int h, PfSeq& sq) {
  const int n = a.len[(long long)a.layer * a.B + b];
  const int qlen = a.q_len[b];
  const int c = a.cap[b];
  const long long base = a.seq_base[b];
  const long long q0 = a.q_start[b];
  const bool ok = n >= 0 && c >= 0 && n <= c && base >= 0 && base + (long long)a.HK * c <= a.rows_per_layer &&
                  qlen >= 0 && qlen <= n && qlen <= a.max_q && n <= a.max_kv && q0 >= 0 && q0 + qlen <= a.q_rows;
  sq.n = n;
  sq.qlen = qlen;
  sq.first = n - qlen;
  sq.q0 = q0;
  sq.row0 = base + (long long)h * c;
  return ok;
}

// ---------------------------------------------------------------------------
// Pass 1: outputs and per-query softmax statistics.
// ---------------------------------------------------------------------------
// The (sequence, KV head, four units) of a block.  Blocks start in the order
// of their indices, so those with the most keys come first: last units first,
// and, when the sequences differ and one lane can hold each (by_length), by
// the 32-key bucket of a block's last key over all sequences.  A block runs
// for up to half a millisecond and the grid is only a few times the 512
// resident blocks, so a long sequence's blocks must not start last (four
// chunks of about 1000 queries over 3001 to 12000 keys: 1012 us a call in unit
// order, 811 us in this one; finding the block takes ten rounds of a wave sum).
// More than 64 sequences, which a wave's lanes cannot hold, keep unit order
// (chunks of 300 queries over 305 to 2948 keys, 4 KV heads: 64 sequences 429 us
// in this order, 66 in unit order 473, 7% more a sequence).
template <int G>
__device__ inline bool pf_block(const PrefillArgs& a, int& b, int& h, int& ub) {
  const int segs = a.B * a.HK;
  const int idx = (int)blockIdx.x;
  if (a.by_length) {
    const int lane = threadIdx.x & (kWave - 1);
    const int bb = min(lane, a.B - 1);  // clamped: lanes past the last sequence repeat it
    const int n = a.len[(long long)a.layer * a.B + bb];
    const int qlen = a.q_len[bb];
    if (!__all(n == __builtin_amdgcn_readfirstlane(n) && qlen == __builtin_amdgcn_readfirstlane(qlen))) {
      // A sequence without queries or with sizes the checks refuse counts as
      // one block, which runs those checks.
      const bool work = n >= 0 && qlen > 0 && qlen <= n && qlen <= a.max_q && n <= a.max_kv;
      const int nb = lane >= a.B ? 0 : work ? ((qlen + 31) / 32 * G + kPfWaves - 1) / kPfWaves : 1;
      // Blocks of this lane's sequence (one head) whose last key is in bucket
      // x or later: those from the unit of the first such tile on.
      auto reach = [&](int x) {
        if (x == 0) return nb;
        if (!work || lane >= a.B || (n - 1) / 32 < x) return 0;
        const int t = max(0, 32 * x - (n - qlen)) / 32;
        return nb - t * G / kPfWaves;
      };
      auto total = [&](int v) { return __builtin_amdgcn_readlane(wave_incl_scan_i32(v), kWave - 1) * a.HK; };
      if (idx >= total(nb)) return false;
      int lo = 0, hi = a.max_kv / 32 + 1;  // buckets >= lo hold block idx, buckets >= hi do not
      while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (total(reach(mid)) > idx)
          lo = mid;
        else
          hi = mid;
      }
      const int above = reach(lo + 1);
      const int here = (reach(lo) - above) * a.HK;
      const int r = idx - total(above);
      const int incl = wave_incl_scan_i32(here);
      b = (int)__builtin_ctzll(__ballot(incl > r));
      const int o = r - __builtin_amdgcn_readlane(incl - here, b);
      h = o % a.HK;
      ub = __builtin_amdgcn_readlane(nb - 1 - above, b) - o / a.HK;
      return true;
    }
  }
  const int seg = idx % segs;
  ub = (int)gridDim.x / segs - 1 - idx / segs;
  b = seg / a.HK;
  h = seg % a.HK;
  return true;
}

// Bound by a SIMD's issue of both units, at a clock that power lowers: at batch
// 8, 2048 tokens, Llama-8B heads, the matrix cores are busy 46% and the vector
// units 50% of the time, next to no time both (two waves a SIMD); both passes do
// 550 GFLOP (P V in two halves, S^T again in pass 2) in 0.62 ms, 0.89 PFLOP/s,
// where an 8192^3 bf16 library product reaches 1.13 to 1.23 on the same data
// distribution (zeros in place of the data: 0.50 ms and 1.70).  16x16x32
// products with 32-key steps took 0.81 ms: twice the LDS reads and softmax
// instructions a flop, and a tile's four waves idled where a group has fewer
// heads.  The V blocks' 64 bytes of padding leave no bank conflicts (with 32
// bytes they take a third of the LDS cycles); two blocks of up to 256 registers
// a lane fit a CU.
template <int D, int G>
__global__ __launch_bounds__(kPfThreads) __attribute__((amdgpu_waves_per_eu(2))) void prefill_fwd_kernel(PrefillArgs a) {
  using Cfg = PfCfg<D>;
  constexpr int KS = Cfg::KS, NT = Cfg::NT, ROWB = Cfg::ROWB, CH = Cfg::CH, STEP = Cfg::STEP;
  static_assert(Cfg::KLOADS % kPfWaves == 0 && Cfg::VLOADS % kPfWaves == 0, "loads split evenly over the waves");
  constexpr int KPW = Cfg::KLOADS / kPfWaves, VPW = Cfg::VLOADS / kPfWaves;  // loads per wave and step
  // Separate arrays, so that the compiler can tell a read of one tile from
  // the direct loads that fill another.
  __shared__ __attribute__((aligned(16))) char ktile0[Cfg::KTILE];
  __shared__ __attribute__((aligned(16))) char ktile1[Cfg::KTILE];
  __shared__ __attribute__((aligned(16))) char vtile0[Cfg::VTILE];
  __shared__ __attribute__((aligned(16))) char vtile1[Cfg::VTILE];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int hh = lane >> 5;  // lane half
  const int s = lane & 31;   // query column
  int b, h, ub;
  if (!pf_block<G>(a, b, h, ub)) return;
  PfSeq sq;
  if (!pf_seq(a, b, h, sq)) {
    if (tid == 0 && ub == 0) atomicOr(a.dev_status, LETHE_DEV_BAD_LAYOUT);
    return;
  }
  const int live = (sq.qlen + 31) / 32;  // tiles with a query
  if (kPfWaves * ub >= live * G) return;
  const int HQ = a.HK * G;
  const int unit = kPfWaves * ub + w;
  const int pt = unit / G, g = unit % G;
  const bool active = pt < live;  // wave-uniform
  const int p0 = sq.first + 32 * pt;
  const int kend = active ? min(sq.n, p0 + 32) : 0;  // keys of this wave
  const int tlast = min((kPfWaves * ub + kPfWaves - 1) / G, live - 1);
  const int kend_blk = min(sq.n, sq.first + 32 * tlast + 32);
  const int nsteps = (kend_blk + STEP - 1) / STEP;
  const char* Kb = reinterpret_cast<const char*>(a.k) + sq.row0 * ROWB;
  const char* Vb = reinterpret_cast<const char*>(a.v) + sq.row0 * ROWB;
  const float sc = a.scale_log2;

  // Queries of this wave's head as the B operand of S^T = K Q^T: lane (hh, s)
  // holds Q[query 32 pt + s][dims 16 kk + 8 hh ..].
  pf_bf16x8_t qb[KS];
  {
    const int i = 32 * pt + s;
    const char* qrow = reinterpret_cast<const char*>(a.q) + ((sq.q0 + i) * HQ + (long long)h * G + g) * ROWB;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      qb[kk] = (active && i < sq.qlen) ? *reinterpret_cast<const pf_bf16x8_t*>(qrow + 32 * kk + 16 * hh) : pf_zero8();
  }

  // This wave's share of a step's tiles: K loads w, w + 4, ... and V loads
  // likewise; the rows of consecutive shares are a constant apart, so one
  // lane offset serves them all.  Rows past the last key of the block (final
  // step only) read that key instead.
  const int krow = (kWave * w + lane) / CH;  // + 256 / CH per load
  const unsigned koff = krow * ROWB + 16 * ((lane % CH) ^ (krow % CH));
  const int vrow = w + Cfg::VLOADS * (lane / Cfg::LPR);  // + kPfWaves per load
  const unsigned voff = vrow * ROWB + 16 * (lane % Cfg::LPR);
  auto issue_k = [&](int st, char* tile) {
    const int j0 = st * STEP;
    if (j0 >= kend_blk) return;
    const char* kt = Kb + (long long)j0 * ROWB;
    pf_lds_char_t* kl = (pf_lds_char_t*)tile + kWave * 16 * w;
    if (j0 + STEP <= kend_blk) {
#pragma unroll
      for (int k = 0; k < KPW; ++k)
        pf_load_lds(kt + k * (kPfThreads / CH) * ROWB, koff, kl + kWave * 16 * kPfWaves * k);
    } else {
      const int last = kend_blk - 1 - j0;
#pragma unroll
      for (int k = 0; k < KPW; ++k)
        pf_load_lds(kt, min(krow + k * (kPfThreads / CH), last) * ROWB + 16 * ((lane % CH) ^ (krow % CH)),
                    kl + kWave * 16 * kPfWaves * k);
    }
  };
  auto issue_v = [&](int st, char* tile) {
    const int j0 = st * STEP;
    if (j0 >= kend_blk) return;
    const char* vt = Vb + (long long)j0 * ROWB;
    pf_lds_char_t* vl = (pf_lds_char_t*)tile + Cfg::VBLK * w;
    if (j0 + STEP <= kend_blk) {
#pragma unroll
      for (int k = 0; k < VPW; ++k) pf_load_lds(vt + k * kPfWaves * ROWB, voff, vl + Cfg::VBLK * kPfWaves * k);
    } else {
      const int last = kend_blk - 1 - j0;
#pragma unroll
      for (int k = 0; k < VPW; ++k)
        pf_load_lds(vt, min(vrow + k * kPfWaves, last) * ROWB + 16 * (lane % Cfg::LPR),
                    vl + Cfg::VBLK * kPfWaves * k);
    }
  };

  const int pos = p0 + s;  // this lane's query position
  float m = kPfNegBig, l = 0.0f, corr = 1.0f;
  float lost = 0.0f;  // last step: sum of the weights less their two halves
  pf_f32x16_t o[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[nt][r] = 0.0f;
  // S^T of a step: lane (hh, s), register r of sub-tile T: key j0 + 32 T +
  // 8 (r / 4) + 4 hh + r % 4, query s.
  pf_f32x16_t sa[2], sb[2];
  auto clear = [&](pf_f32x16_t (&x)[2]) {
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int r = 0; r < 16; ++r) x[T][r] = 0.0f;
  };
  auto qk = [&](pf_f32x16_t (&x)[2], const char* kt, int kk) {
#pragma unroll
    for (int T = 0; T < 2; ++T) {
      const pf_bf16x8_t kr = *reinterpret_cast<const pf_bf16x8_t*>(kt + 16 * Cfg::kslot(32 * T + s, 2 * kk + hh));
      x[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr, qb[kk], x[T], 0, 0, 0);
    }
  };
  // Steps wholly below the diagonal (every key precedes every query of the
  // unit and is live) skip the mask.
  auto mask = [&](pf_f32x16_t (&x)[2], int j0) {
    if (j0 + STEP - 1 > p0 || j0 + STEP > kend) {
      asm volatile("");  // keeps the mask behind a branch
      const int lim = min(pos, kend - 1) - j0 - 4 * hh;
#pragma unroll
      for (int T = 0; T < 2; ++T)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (32 * T + 8 * (r >> 2) + (r & 3) > lim) x[T][r] = -INFINITY;
    }
  };
  auto row_max = [&](const pf_f32x16_t (&x)[2]) {
    float mx = fmaxf(x[0][0], x[1][0]);
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(fmaxf(mx, x[0][r]), x[1][r]);
    return mx;
  };
  // V^T operand of keys 16 mm .. + 15 and dims 32 nt .. through the
  // transposing LDS read: lane i of a 16-lane group points at row 4 hh + i / 4
  // (and 8 rows further), 4 columns from 32 nt + 16 (group mod 2) + 4 (i mod 4).
  auto v_operand = [&](const char* vtile, int mm, int nt) {
    const pf_lds_char_t* vt = (const pf_lds_char_t*)vtile;
    const int vr = 16 * mm + 4 * hh + ((lane & 15) >> 2);
    const int col = (32 * nt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
    const pf_bf16x4_t a0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((pf_lds_bf16x4_t*)(vt + Cfg::vaddr(vr, col)));
    const pf_bf16x4_t a1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((pf_lds_bf16x4_t*)(vt + Cfg::vaddr(vr + 8, col)));
    return __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // Once the running maxima settle most steps leave every lane's correction
  // at exactly 1; the wave then skips the rescale.
  auto rescale = [&]() {
    if (__any(corr != 1.0f)) {
      l *= corr;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[nt][r] *= corr;
    }
  };
  auto new_max = [&](const pf_f32x16_t (&x)[2]) {
    const float mnew = fmaxf(m, pf_max_halves(row_max(x)) * sc);
    corr = hw_exp2(m - mnew);
    m = mnew;
  };
  // P of 16 keys in bf16 high and low parts: registers 8 (mm % 2) .. of
  // sub-tile mm / 2 are the B operand of those keys in the order (j < 4:
  // 4 hh + j, else 8 + 4 hh + j - 4) that the V^T operand follows.  A wave's
  // last step also sums what the two halves miss (up to 2^-18 of a weight), and
  // the output is divided by the sum of the weights it was made of: a row whose
  // weight lies on a few keys then keeps their exact ratio.  Errors against 64
  // bits, batch 8 x 2048 and three prompts of 77 to 421 rows: 1.686e-6 and
  // 1.510e-6 without, 1.663e-6 and 1.465e-6 with it (0.2% of the time); every
  // step counted, 1.652e-6 and 1.456e-6 (6%).
  float psum[2] = {0.0f, 0.0f};
  auto weights = [&](const pf_f32x16_t (&x)[2], int mm, pf_bf16x8_t& ph, pf_bf16x8_t& pl, auto last) {
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
      const float pa = hw_exp2(fmaf(x[mm >> 1][8 * (mm & 1) + j], sc, -m));
      const float pb = hw_exp2(fmaf(x[mm >> 1][8 * (mm & 1) + j + 1], sc, -m));
      psum[0] += pa;
      psum[1] += pb;
      const pf_bf16x2_t hi = __builtin_convertvector((pf_f32x2_t{pa, pb}), pf_bf16x2_t);
      const unsigned hb = __builtin_bit_cast(unsigned, hi);
      const float ra = pa - __uint_as_float(hb << 16), rb = pb - __uint_as_float(hb & 0xffff0000u);
      const pf_bf16x2_t lo = __builtin_convertvector((pf_f32x2_t{ra, rb}), pf_bf16x2_t);
      if constexpr (last) {
        const unsigned lb = __builtin_bit_cast(unsigned, lo);
        lost += (ra - __uint_as_float(lb << 16)) + (rb - __uint_as_float(lb & 0xffff0000u));
      }
      ph[j] = hi[0];
      ph[j + 1] = hi[1];
      pl[j] = lo[0];
      pl[j + 1] = lo[1];
    }
  };
  auto pv = [&](const char* vtile, int mm, const pf_bf16x8_t& ph, const pf_bf16x8_t& pl) {
    pf_bf16x8_t av[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) av[nt] = v_operand(vtile, mm, nt);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[nt], ph, o[nt], 0, 0, 0);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[nt], pl, o[nt], 0, 0, 0);
  };
  // A step of this wave that is not its last: the softmax weights and P V of
  // step st, whose S^T is in sx, interleaved with S^T of step st + 1 into sn
  // (K runs one tile ahead of V), so that the matrix cores work on both
  // products while the weights are formed.
  auto body = [&](int st, pf_f32x16_t (&sx)[2], pf_f32x16_t (&sn)[2], const char* knext, const char* vcur) {
    rescale();
    clear(sn);
    psum[0] = psum[1] = 0.0f;
    pf_bf16x8_t ph, pl, nh, nl;
    weights(sx, 0, ph, pl, std::false_type());
#pragma unroll
    for (int kk = 0; kk < KS / 4; ++kk) qk(sn, knext, kk);
#pragma unroll
    for (int mm = 1; mm < 4; ++mm) {
      weights(sx, mm, nh, nl, std::false_type());
#pragma unroll
      for (int kk = mm * KS / 4; kk < (mm + 1) * KS / 4; ++kk) qk(sn, knext, kk);
      pv(vcur, mm - 1, ph, pl);
      ph = nh;
      pl = nl;
    }
    l += psum[0] + psum[1];
    mask(sn, (st + 1) * STEP);
    pv(vcur, 3, ph, pl);
    new_max(sn);
  };
  // This wave's last step.  Rows past its keys that another wave's tile
  // brought in have weight 0, and count as 0 so that an infinity there stays
  // out of the sum.
  auto last_body = [&](int st, const pf_f32x16_t (&sx)[2], const char* vcur) {
    rescale();
    psum[0] = psum[1] = 0.0f;
#pragma unroll
    for (int mm = 0; mm < 4; ++mm) {
      pf_bf16x8_t ph, pl;
      weights(sx, mm, ph, pl, std::true_type());
      if constexpr (G % kPfWaves == 0) {
        pv(vcur, mm, ph, pl);
      } else {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          pf_bf16x8_t av = v_operand(vcur, mm, nt);
#pragma unroll
          for (int j = 0; j < 8; ++j)
            if (st * STEP + 16 * mm + 4 * hh + 8 * (j >> 2) + (j & 3) >= kend) av[j] = (__bf16)0.0f;
          o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, ph, o[nt], 0, 0, 0);
          o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, pl, o[nt], 0, 0, 0);
        }
      }
    }
    l += psum[0] + psum[1];
  };

  // At step st, K of step st + 2 and V of step st + 1 are on their way into
  // the buffers that step st - 1 has used.  Each wave waits for its own loads
  // (the barrier alone would not); the barrier then makes every wave's visible
  // and guarantees that the buffers to fill have been read by all.
  auto advance = [&](int st, char* kfill, char* vfill) {
    wait_vmem();
    __syncthreads();
    issue_k(st + 2, kfill);
    issue_v(st + 1, vfill);
  };
  issue_k(0, ktile0);
  issue_k(1, ktile1);
  issue_v(0, vtile0);
  wait_vmem();
  __syncthreads();
  const int own = (kend + STEP - 1) / STEP;  // steps of this wave
  clear(sa);
  if (active) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qk(sa, ktile0, kk);
    mask(sa, 0);
    new_max(sa);
  }
  int st = 0;
  for (; st + 2 < own; st += 2) {
    advance(st, ktile0, vtile1);
    body(st, sa, sb, ktile1, vtile0);
    advance(st + 1, ktile1, vtile0);
    body(st + 1, sb, sa, ktile0, vtile1);
  }
  if (st + 1 < own) {
    advance(st, ktile0, vtile1);
    body(st, sa, sb, ktile1, vtile0);
    ++st;
    sa[0] = sb[0];
    sa[1] = sb[1];
  }
  if (active) {
    advance(st, (st & 1) ? ktile1 : ktile0, (st & 1) ? vtile0 : vtile1);
    last_body(st, sa, (st & 1) ? vtile1 : vtile0);
    ++st;
  }
  for (; st < nsteps; ++st) advance(st, (st & 1) ? ktile1 : ktile0, (st & 1) ? vtile0 : vtile1);
  if (!active) return;

  // l and lost are split over the two lane halves of a query column; m is
  // common.  The statistics keep the exact sum.
  l += __shfl_xor(l, 32);
  lost += __shfl_xor(lost, 32);
  const int i = 32 * pt + s;
  if (i >= sq.qlen) return;
  const float inv = 1.0f / l, winv = 1.0f / (l - lost);
  float* orow = a.out + ((sq.q0 + i) * HQ + (long long)h * G + g) * D;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int r = 0; r < 16; r += 4)
      *reinterpret_cast<float4*>(orow + 32 * nt + 2 * r + 4 * hh) =
          make_float4(o[nt][r] * winv, o[nt][r + 1] * winv, o[nt][r + 2] * winv, o[nt][r + 3] * winv);
  if (hh == 0)
    *reinterpret_cast<float2*>(a.stat + 2 * ((long long)(h * G + g) * a.q_rows + sq.q0 + i)) = make_float2(m, inv);
}

// ---------------------------------------------------------------------------
// Pass 2: importance seeding, key-major.
// ---------------------------------------------------------------------------
// A block is KW key waves of 32 NS keys each times IG item groups: group ig
// takes the work items (tile of 32 queries, head) ig, ig + IG, ... and keeps
// its own double-buffered query tile.  A weight costs a multiply-add, an exp2
// and a multiply-add against 16 matrix-core cycles a lane, so the pass needs
// waves to overlap the two: 32 keys a wave hold 116 registers, four waves a
// SIMD, where 64 keys held 190.  At batch 8, 2048 tokens it takes 0.18 ms, the
// vector units busy 59% and the matrix cores 35% of it.
template <int D, int G, int NS, int KW, int IG>
__global__ __launch_bounds__(kWave * KW * IG) __attribute__((amdgpu_waves_per_eu(KW * IG / 4))) void
    prefill_score_kernel(PrefillArgs a) {
  using Cfg = PfCfg<D>;
  constexpr int KS = Cfg::KS, ROWB = Cfg::ROWB, CH = Cfg::CH;
  constexpr int QTILE = 32 * ROWB;
  constexpr int QLOADS = QTILE / (kWave * 16);
  static_assert(QLOADS % KW == 0, "query loads split evenly over the group's waves");
  constexpr int LPW = QLOADS / KW;
  constexpr int KEYS = 32 * NS * KW;  // keys per block
  __shared__ __attribute__((aligned(16))) char buf0[IG * QTILE];
  __shared__ __attribute__((aligned(16))) char buf1[IG * QTILE];
  __shared__ float sums[IG][KEYS];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int kw = w % KW, ig = w / KW;
  const int hh = lane >> 5;
  const int s = lane & 31;
  const int b = (int)blockIdx.x / a.HK, h = (int)blockIdx.x % a.HK;
  const long long kb = blockIdx.y + (long long)gridDim.y * blockIdx.z;  // low keys (most queries) first
  PfSeq sq;
  if (!pf_seq(a, b, h, sq)) return;  // flagged by the forward pass
  if (sq.qlen == 0 || kb * KEYS >= sq.n) return;
  const int kblk0 = (int)kb * KEYS;
  const int HQ = a.HK * G;
  const int j0w = kblk0 + 32 * NS * kw;
  const char* Kb = reinterpret_cast<const char*>(a.k) + sq.row0 * ROWB;
  const float sc = a.scale_log2;

  // This wave's keys as the A operand (row 32 T + s, dims 16 kk + 8 hh ..).
  pf_bf16x8_t kr[NS][KS];
#pragma unroll
  for (int T = 0; T < NS; ++T) {
    const int row = min(j0w + 32 * T + s, sq.n - 1);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      kr[T][kk] = *reinterpret_cast<const pf_bf16x8_t*>(Kb + (long long)row * ROWB + 32 * kk + 16 * hh);
  }

  // Work items: (tile of 32 queries, head) for every tile holding a position
  // at or after the block's first key.
  const int it0 = max(0, kblk0 - sq.first) / 32;
  const int nitems = ((sq.qlen + 31) / 32 - it0) * G;
  const int qrow = (kWave * kw + lane) / CH;  // + 64 KW / CH per load
  float2 st_next = make_float2(0.0f, 0.0f);
  auto issue = [&](int item, char* buf) {
    if (item >= nitems) return;
    const int it = it0 + item / G, g = item % G;
    const char* src = reinterpret_cast<const char*>(a.q) + ((sq.q0 + 32 * it) * HQ + (long long)h * G + g) * ROWB;
    const int last = sq.qlen - 1 - 32 * it;  // queries past it read it instead
#pragma unroll
    for (int k = 0; k < LPW; ++k) {
      const int r = qrow + k * (kWave * KW / CH);
      const int c = (lane % CH) ^ (r % CH);
      pf_load_lds(src, (unsigned)(min(r, last) * HQ) * ROWB + 16 * c,
                  (pf_lds_char_t*)buf + ig * QTILE + kWave * 16 * (kw + KW * k));
    }
    st_next = *reinterpret_cast<const float2*>(
        a.stat + 2 * ((long long)(h * G + g) * a.q_rows + sq.q0 + 32 * it + min(s, last)));
  };

  float acc[NS][16];
#pragma unroll
  for (int T = 0; T < NS; ++T)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[T][r] = 0.0f;

  auto compute = [&](int item, const char* buf, float2 qs) {
    if (item >= nitems || j0w >= sq.n) return;
    const int it = it0 + item / G;
    const int pos0 = sq.first + 32 * it;  // position of the tile's first query
    if (pos0 + 31 < j0w) return;          // every query precedes this wave's keys
    const char* qt = buf + ig * QTILE;
    pf_bf16x8_t qv[KS];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      qv[kk] = *reinterpret_cast<const pf_bf16x8_t*>(qt + 16 * Cfg::kslot(s, 2 * kk + hh));
    pf_f32x16_t sacc[NS];
#pragma unroll
    for (int T = 0; T < NS; ++T) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sacc[T][r] = 0.0f;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        sacc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[T][kk], qv[kk], sacc[T], 0, 0, 0);
    }
    // Tiles whose every query is live and follows every key skip the mask
    // (a masked weight is left out, whatever its query's statistics hold).
    if (j0w + 32 * NS - 1 > pos0 || 32 * (it + 1) > sq.qlen) {
      const int lim = 32 * it + s < sq.qlen ? pos0 + s - j0w - 4 * hh : -1;
#pragma unroll
      for (int T = 0; T < NS; ++T)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = hw_exp2(fmaf(sacc[T][r], sc, -qs.x)) * qs.y;
          acc[T][r] += 32 * T + 8 * (r >> 2) + (r & 3) > lim ? 0.0f : p;
        }
    } else {
#pragma unroll
      for (int T = 0; T < NS; ++T)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[T][r] = fmaf(hw_exp2(fmaf(sacc[T][r], sc, -qs.x)), qs.y, acc[T][r]);
    }
  };

  issue(ig, buf0);
  const int rounds = (nitems + IG - 1) / IG;
  for (int x = 0; x < rounds; x += 2) {
    wait_vmem();
    __syncthreads();
    float2 qs = st_next;
    issue((x + 1) * IG + ig, buf1);
    compute(x * IG + ig, buf0, qs);
    if (x + 1 >= rounds) break;
    wait_vmem();
    __syncthreads();
    qs = st_next;
    issue((x + 2) * IG + ig, buf0);
    compute((x + 1) * IG + ig, buf1, qs);
  }

  // Sum over the 32 query columns: each exchange halves the keys a lane
  // holds, until lane s holds key register s / 2.
#pragma unroll
  for (int T = 0; T < NS; ++T) {
#pragma unroll
    for (int half = 8; half >= 1; half /= 2) {
      const bool up = (s & (2 * half)) != 0;
#pragma unroll
      for (int r = 0; r < half; ++r) {
        const float mine = up ? acc[T][r + half] : acc[T][r];
        const float give = up ? acc[T][r] : acc[T][r + half];
        acc[T][r] = mine + __shfl_xor(give, 2 * half);
      }
    }
    const float v = acc[T][0] + __shfl_xor(acc[T][0], 1);
    const int r = s >> 1;
    if ((s & 1) == 0) sums[ig][32 * (NS * kw + T) + 8 * (r >> 2) + 4 * hh + (r & 3)] = v;
  }
  __syncthreads();
  for (int j = tid; j < KEYS && kblk0 + j < sq.n; j += kWave * KW * IG) {
    float t = sums[0][j];
#pragma unroll
    for (int x = 1; x < IG; ++x) t += sums[x][j];
    a.score[sq.row0 + kblk0 + j] += t;
  }
}

// One block per segment (x) and key block (y, then z).  max_kv is only a bound:
// a grid of one dimension would be refused from 2^32 threads on (1024 segments
// and a bound of 2^20 rows), whatever the lengths are.
template <int D, int G, int NS, int KW, int IG>
lethe_status launch_score(const PrefillArgs& a, unsigned segs, hipStream_t s) {
  constexpr long long kKeys = 32 * NS * KW, kMaxY = 32768;
  const long long kblocks = (a.max_kv + kKeys - 1) / kKeys;
  const unsigned y = (unsigned)std::min(kblocks, kMaxY), z = (unsigned)((kblocks + y - 1) / y);
  hipLaunchKernelGGL((prefill_score_kernel<D, G, NS, KW, IG>), dim3(segs, y, z), dim3(kWave * KW * IG), 0, s, a);
  return hipGetLastError() == hipSuccess ? LETHE_OK : LETHE_ERR_HIP;
}

template <int D, int G>
lethe_status launch_prefill_dg(const PrefillArgs& args, hipStream_t s) {
  PrefillArgs a = args;
  // The bounds a caller passes may be loose (INT32_MAX): no sequence that
  // passes the kernels' checks has more queries than there are query rows or
  // more rows than a segment of this layer can have.
  a.max_q = (int32_t)std::min<int64_t>(a.max_q, std::max<int64_t>(a.q_rows, 1));
  a.max_kv = (int32_t)std::min<int64_t>(a.max_kv, a.rows_per_layer / a.HK);
  const long long segs = (long long)a.B * a.HK;
  const long long nq = (a.max_q + 31LL) / 32;
  const long long fwd_blocks = segs * ((nq * G + kPfWaves - 1) / kPfWaves);
  // A launch's threads in x must stay below 2^32; refused before the first one
  // (from 256 segments on the score blocks have 512 threads).
  if (fwd_blocks * kPfThreads > 0xffffffffLL || segs * 512 > 0xffffffffLL) return LETHE_ERR_UNSUPPORTED;
  a.by_length = a.B > 1 && a.B <= kWave && fwd_blocks > kPfResident;
  if (fwd_blocks > 0) {
    hipLaunchKernelGGL((prefill_fwd_kernel<D, G>), dim3((unsigned)fwd_blocks), dim3(kPfThreads), 0, s, a);
    if (hipGetLastError() != hipSuccess) return LETHE_ERR_HIP;
  }
  const long long wide = segs * ((a.max_kv + 127LL) / 128);
  if (wide == 0 || fwd_blocks == 0) return LETHE_OK;
  // 128 keys a block where those blocks fill the chip's 256 CUs, else 64 keys
  // and eight item groups, one block a CU (24 segments of 77 to 421 rows: 12 us
  // against 64 us with 256 keys a block).  Whole calls, 64 against 128 keys:
  // prompts of 1000 to 3000 rows, 64 to 192 blocks of 128, 28 to 22% less; 256
  // blocks 5 to 20% less (the first keys meet every query, and their blocks
  // last); 512 and 1024 blocks 7 to 12% more.  Chunks of 200 queries, whose
  // blocks are alike: 64 and 96 blocks 8 to 9% less, 136 alike, 160 to 256 5 to
  // 12% more, 1024 29% more.  The line lies between the two.
  if (wide >= 256) return launch_score<D, G, 1, 4, 2>(a, (unsigned)segs, s);
  return launch_score<D, G, 1, 2, 8>(a, (unsigned)segs, s);
}

template <int D>
lethe_status launch_prefill_d(const PrefillArgs& a, int G, hipStream_t s) {
  switch (G) {
    case 1: return launch_prefill_dg<D, 1>(a, s);
    case 2: return launch_prefill_dg<D, 2>(a, s);
    case 3: return launch_prefill_dg<D, 3>(a, s);
    case 4: return launch_prefill_dg<D, 4>(a, s);
    case 5: return launch_prefill_dg<D, 5>(a, s);
    case 6: return launch_prefill_dg<D, 6>(a, s);
    case 7: return launch_prefill_dg<D, 7>(a, s);
    case 8: return launch_prefill_dg<D, 8>(a, s);
    default: return LETHE_ERR_UNSUPPORTED;
  }
}

}  // namespace

lethe_status launch_prefill(const PrefillArgs& a, int D, int G, hipStream_t s) {
  if (D == 128) return launch_prefill_d<128>(a, G, s);
  if (D == 64) return launch_prefill_d<64>(a, G, s);
  return LETHE_ERR_UNSUPPORTED;
}

}  // namespace lethe
