// Temperature / nucleus (top-p) sampling with caller-supplied uniforms.
//
// RL rollouts sample their actions rather than taking the argmax (paper:
// Background, "RL Post-Training Workflow"); the paper does not state the
// sampler, so this is the common temperature + top-p rule, defined so that
// every decision is exact integer arithmetic after one exponential:
//
//   e_v = exp((z_v - max z) / T)            (fp64)
//   q_v = rint(e_v * 2^40)                  (integer mass, 0 .. 2^40)
//   S   = sum_v q_v
//   nucleus: the shortest prefix of the tokens ordered by (q desc, index asc)
//            whose mass reaches T_p = ceil(p24 * S / 2^24), p24 = rint(top_p * 2^24)
//   Z   = nucleus mass, target = floor(u24 * Z / 2^24), u24 = floor(u * 2^24)
//   token = the first nucleus token, in index order, whose running nucleus
//           mass exceeds target.
//
// The threshold key kappa (the largest key with mass{q >= kappa} >= T_p) is
// found in the order of x = (z - max z)/T, in which the masses are monotone:
//   1. the row maximum;
//   2. every token's mass into a histogram over x (16 bins an octave, 64-bit
//      integer LDS atomics, so their order does not matter); its total is S
//      and the bin that crosses T_p holds the threshold;
//   3. a second pass sums, per index block, the masses above that bin and
//      lists the bin's own tokens (a few hundred of 128K);
//   4. kappa, the ties at kappa that join the nucleus (lowest indices first)
//      and each block's nucleus mass follow from the list alone;
//   5. only the index block that holds the target is walked token by token.
// So a row is read three times and each token's exponential is evaluated once,
// plus once more for nucleus members; a radix select over the keys themselves
// re-evaluates it in every round whose digit range holds most of the row.  At
// 128256 logits N(0, 9), T 0.8, top_p 0.95, against that radix select: 256 rows
// (one work group each) 100 us instead of 323, 16 rows (the split form) 34 us
// instead of 135.  What is left at 256 rows: the three passes (18 us at the HBM
// rate, ~45 of fp64 arithmetic, ~30 for the second pass) and ~10 of decisions.
// With top_p = 1 the nucleus is every token of nonzero mass: steps 2 to 4
// reduce to the per-block masses.
//
// The list holds 8192 tokens of a row.  A bin is T ln2 / 16 wide in logits, so a row
// of deviation s has 1.7% of its tokens there with s = T and more with a smaller s;
// at 128256 tokens the list holds out to s = 0.3 T or so.  A wider bin, many equal
// logits, or a threshold so deep (masses below 64) that one key spans several bins
// takes a second histogram, over the keys of the bin (cut_bin), whose pass also
// gives each block's whole mass, so that the last pass evaluates the tokens at the
// threshold and below instead of the members.  us, radix select / this: 256 rows
// N(0, 0.0004) 296 / 213, all equal 411 / 184; 16 rows 130 / 81 and 143 / 105.
#include "hip_common.h"
#include "kernels.h"

#include <algorithm>
#include <climits>
#include <mutex>

namespace pdec {

namespace {

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kBins = 1024;        // histogram bins, one per thread of a row's group
constexpr double kOctave = 16.0;   // step 2: bins per factor of two of the mass (670 of them)
constexpr int kMaxBlocks = 128;    // index blocks of a row
constexpr int kSlab = 512;         // tokens a wave holds at a time, 8 per lane
constexpr int kListCap = 8192;     // threshold-bin tokens held in LDS
constexpr double kMinX = -28.5;    // below it the mass rounds to 0
constexpr double kLn2 = 0.69314718055994530942;
constexpr double kMinKey = 64.0;   // step 3 needs one key to stay within about one bin
typedef unsigned __int128 u128;

// Length of a row's index blocks (a multiple of 256): at most kMaxBlocks of
// them, 1024 tokens each for the 128256-token vocabulary.
__host__ __device__ __forceinline__ int block_len(int V) {
  const int64_t b = ((int64_t)V + kMaxBlocks - 1) / kMaxBlocks;
  return (int)((b + 255) / 256 * 256);
}

// Integer mass at x <= 0 (NaN: 0).  Below x = -28.5 the exponential is under
// 2^-41 and the mass rounds to exactly 0.  Adding 2^52 rounds e * 2^40 to an
// integer (to nearest even, as rint) and leaves it in the mantissa bits.
__device__ __forceinline__ uint64_t mass_at(double x) {
  if (!(x >= kMinX)) return 0;
  return __double_as_longlong(__builtin_fma(exp(x), 0x1p40, 0x1p52)) - 0x4330000000000000ull;
}

__device__ __forceinline__ uint64_t lane_u64(uint64_t v, int lane) {  // lane uniform
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
  return ((uint64_t)hi << 32) | lo;
}

// Inclusive scan over the wave, all lanes active: shifts within the rows of 16 lanes,
// then row ends broadcast to the rows behind them (DPP moves: no LDS permutes, and no
// lane addresses kept in registers).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t v) {  // 0 where there is no source lane
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xf, false);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t wave_scan_incl(uint64_t v) {
  v += dpp_u64<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8
  v += dpp_u64<0x112, 0xf>(v);
  v += dpp_u64<0x114, 0xf>(v);
  v += dpp_u64<0x118, 0xf>(v);
  v += dpp_u64<0x142, 0xa>(v);  // row_bcast:15 to rows 1 and 3
  v += dpp_u64<0x143, 0xc>(v);  // row_bcast:31 to rows 2 and 3
  return v;
}
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) { return lane_u64(wave_scan_incl(v), 63); }

// A value that is the same in all lanes (read from LDS), in scalar registers.
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float scalar(float v) { return __int_as_float(scalar(__float_as_int(v))); }
__device__ __forceinline__ uint64_t scalar(uint64_t v) {
  return ((uint64_t)(uint32_t)scalar((int)(v >> 32)) << 32) | (uint32_t)scalar((int)(uint32_t)v);
}
__device__ __forceinline__ double scalar(double v) {
  return __longlong_as_double((int64_t)scalar((uint64_t)__double_as_longlong(v)));
}

// What follows from the temperature T, computed on the host (kernel arguments stay in
// scalar registers, divisions of the GPU do not).
struct Scale {
  double inv_t;  // 1 / T
  double dmin;   // -29 T: logits this far below the maximum have no mass
  double c1;     // bins per unit of logit
  float t;       // T, at most 10^36
};

// threadIdx.x, made anew: what is computed from it (LDS addresses) is not kept in
// registers from one pass over the row to the next.
__device__ __forceinline__ int thread_id() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

__device__ __forceinline__ uint64_t zero_u64() {  // likewise
  uint32_t z = 0;
  asm volatile("" : "+v"(z));
  return ((uint64_t)z << 32) | z;
}

// One row as a wave reads it: 8 tokens per lane of a slab of kSlab tokens.
// VEC: 16-byte loads (the row starts 16-byte aligned and V % 4 == 0).
template <bool VEC>
struct Row {
  const float* z;
  int V, blen, nb;
  double m, inv_t;
  // Not to be fused into what a caller does with it: two callers have to see
  // the same x for the same logit.
  __device__ __forceinline__ double x(float v) const {
#pragma clang fp contract(off)
    return ((double)v - m) * inv_t;
  }
  // The lane's tokens of the slab at token `at`, loads only: indices past the
  // row's end read its last tokens, and mask() turns them into -inf once the
  // loads are waited for.
  __device__ __forceinline__ void load(int at, int lane, float (&v)[8]) const {
    // A uniform base and 32-bit byte offsets: one register per address.
    const char* base = (const char*)(z + at);
    const uint32_t last = (uint32_t)min(V - 1 - at, kSlab + 3);
#pragma unroll
    for (int u = 0; u < 8; u += VEC ? 4 : 1) {
      if constexpr (VEC) {
        const float4 f = *(const float4*)(base + 4 * min(u * 64u + 4 * lane, last - 3));
        v[u] = f.x;
        v[u + 1] = f.y;
        v[u + 2] = f.z;
        v[u + 3] = f.w;
      } else {
        v[u] = *(const float*)(base + 4 * min(u * 64u + lane, last));
      }
    }
  }
  // n: tokens of the slab that belong to the block.
  __device__ __forceinline__ void mask(int n, int lane, const float (&w)[8], float (&v)[8]) const {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      v[u] = (VEC ? (u & 4) * 64 + 4 * lane : u * 64 + lane) < n ? w[u] : -INFINITY;
  }
  // Index within the slab of a lane's element k of part `part`.
  __device__ __forceinline__ int offset(int part, int k, int lane) const {
    return part * 256 + (VEC ? 4 * lane + k : k * 64 + lane);
  }
  // f(block, first token, part, four of the lane's values, whether the block
  // ends there) for both parts of every slab of blocks b, b + step, .. below
  // b1, the next slab's loads in flight meanwhile.  The parts run through one
  // copy of f's code: a launch runs it a few times per wave, and fetching 16
  // unrolled copies of it cost more than running them (split_members: 20 us
  // against 6).
  template <typename F>
  __device__ __forceinline__ void slabs(int b, int b1, int step, int lane, F&& f) const {
    if (b >= b1) return;
    asm volatile("" : "+s"(b));  // addresses are made here, not kept from one pass to the next
    int o = 0, n = min(blen, V - b * blen);
    float v[8], w[8];
    load(b * blen, lane, w);
    mask(n, lane, w, v);
    wait_vmem<0>();  // nothing but the next slab is in flight inside the loop
    for (;;) {
      const bool end = o + kSlab >= n;
      const int b2 = end ? b + step : b, o2 = end ? 0 : o + kSlab;
      const bool more = b2 < b1;
      load(more ? b2 * blen + o2 : b * blen + o, lane, w);  // the last slab again at the end
#pragma unroll 1
      for (int part = 0; part < 2; ++part) {
        float h[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) h[k] = part ? v[4 + k] : v[k];
        f(b, b * blen + o, part, h, end && part);
      }
      if (!more) break;
      b = b2;
      o = o2;
      n = min(blen, V - b * blen);
      mask(n - o, lane, w, v);
    }
  }
};

template <bool VEC>
__device__ __forceinline__ Row<VEC> make_row(int V, const float* logits, int b, const Scale& sc) {
  Row<VEC> r;
  r.z = logits + (int64_t)b * V;
  r.V = V;
  r.blen = block_len(V);
  r.nb = (V - 1) / r.blen + 1;
  r.m = 0.0;
  r.inv_t = sc.inv_t;
  return r;
}

// The masses of a pass over a whole row.  mass_at takes about 60 operations in
// one dependent chain (the pass took 51 us for 256 rows, one per CU, with or
// without its LDS atomics).  Here, with the row's scale folded into one
// constant and 2^(j/16) * 2^40 in a 16-entry LDS table (entries in distinct
// banks): t = (z - max z) * 16 / (T ln 2) = n + r, |r| <= 1/2, and
//   e * 2^40 = 2^(n >> 4) * table[n & 15] * exp(r ln2 / 16),
// the last factor a Taylor polynomial of degree 6 (next term (ln2/32)^7 / 7! =
// 4.5e-16).  With the roundings the product is within (1.5e-15 + 4e-16 |x|) of
// exp(x) * 2^40, relatively, |x| <= 29, so below 1.4e-14; where that could
// change the rounding to an integer (a distance under 4e-14 of the value to a
// half: every 10^6th token at e = 2^-15), mass_at decides.  The keys are
// therefore mass_at's, bit for bit.  -n also numbers the histogram's bins.
struct FastMass {
  double m;
  Scale c;
  const double* table;  // LDS
};
__device__ __forceinline__ void fill_table(double* table) {  // then a barrier
  if (threadIdx.x < 16) table[threadIdx.x] = exp2((double)threadIdx.x / 16.0 + 40.0);
}
__device__ __forceinline__ FastMass make_fast(double m, const Scale& sc, const double* table) {
  return {m, sc, table};
}
// The keys of N logits (0 below x = -29 and for NaN) and their bins; bit k of
// the result is set where mass_at has to decide.  The N chains of dependent fp64
// operations run side by side.
template <int N>
__device__ __forceinline__ uint32_t fast_mass(const FastMass& fm, const float (&z)[N],
                                              uint64_t (&q)[N], int (&bin)[N]) {
  constexpr double kRound = 6755399441055744.0;  // 1.5 * 2^52: n in the low mantissa bits
  constexpr double a = kLn2 / kOctave;
  constexpr double coef[6] = {a * a * a * a * a / 120.0, a * a * a * a / 24.0, a * a * a / 6.0,
                              a * a / 2.0, a, 1.0};
  double r[N], p[N], tb[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double d = fmax((double)z[k] - fm.m, fm.c.dmin);
    const double un = __builtin_fma(d, fm.c.c1, kRound);
    const int n = (int)(uint32_t)__double_as_longlong(un);
    bin[k] = -n;
    const int64_t t = __double_as_longlong(fm.table[n & 15]);
    tb[k] = __longlong_as_double(t + ((int64_t)(n >> 4) << 52));
    r[k] = __builtin_fma(d, fm.c.c1, -(un - kRound));
    p[k] = a * a * a * a * a * a / 720.0;
  }
#pragma unroll
  for (int c = 0; c < 6; ++c)
#pragma unroll
    for (int k = 0; k < N; ++k) p[k] = __builtin_fma(p[k], r[k], coef[c]);
  uint32_t close = 0;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double v = tb[k] * p[k];
    const double w = v + 0x1p52;
    const double off = fabs(v - (w - 0x1p52));  // exact; 1/2 at a tie
    close |= __builtin_fma(v, 4e-14, off) >= 0.5 ? 1u << k : 0u;
    q[k] = (uint64_t)__double_as_longlong(w) & 0xFFFFFFFFFFFFFull;
  }
  return close;
}

// Element k of a lane's four values, k different per lane.
template <typename T>
__device__ __forceinline__ T pick4(const T (&v)[4], int k) {
  const T a = k & 1 ? v[1] : v[0], b = k & 1 ? v[3] : v[2];
  return k & 2 ? b : a;
}

// Step 2 for a part of a slab: masses into hist by bin.  Runs of equal bins in a lane
// are added up first, so that a row of equal logits does not send four atomics
// per lane to one address.
template <bool VEC>
__device__ __forceinline__ void slab_hist(const Row<VEC>& row, const FastMass& fm, const float (&v)[4],
                                          uint64_t* hist) {
  uint64_t q[4];
  int bin[4];
  uint32_t redo = fast_mass<4>(fm, v, q, bin);
  if (__any(redo != 0)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = redo >> k & 1 ? 0 : q[k];
    while (redo) {
      const int k = __ffs(redo) - 1;
      redo &= redo - 1;
      const uint64_t e = mass_at(row.x(pick4(v, k)));
      if (e) atomicAdd((unsigned long long*)&hist[pick4(bin, k)], e);
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k < 3 && bin[k] == bin[k + 1]) q[k + 1] += q[k];
    else if (q[k]) atomicAdd((unsigned long long*)&hist[bin[k]], q[k]);
  }
}

// Sum of the masses of the lane's tokens in mask, of which a lane usually has
// none or one: each lane evaluates its own next one.
template <bool VEC>
__device__ __forceinline__ uint64_t slab_mass(const Row<VEC>& row, const FastMass& fm,
                                              const float (&v)[4], uint32_t mask) {
  uint64_t sum = 0;
  while (mask) {
    const float z[1] = {pick4(v, __ffs(mask) - 1)};
    mask &= mask - 1;
    uint64_t q[1];
    int bin[1];
    if (__builtin_expect(fast_mass<1>(fm, z, q, bin), 0)) q[0] = mass_at(row.x(z[0]));
    sum += q[0];
  }
  return sum;
}

// Sum of all four masses.
template <bool VEC>
__device__ __forceinline__ uint64_t slab_mass_all(const Row<VEC>& row, const FastMass& fm,
                                                  const float (&v)[4]) {
  uint64_t q[4];
  int bin[4];
  uint32_t redo = fast_mass<4>(fm, v, q, bin);
  uint64_t sum = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) sum += redo >> k & 1 ? 0 : q[k];
  while (redo) {
    sum += mass_at(row.x(pick4(v, __ffs(redo) - 1)));
    redo &= redo - 1;
  }
  return sum;
}

// The bounds of step 3.  Logits at or above z1 are above every key of the
// threshold bin: z1 lies past the bin's upper edge by what one key spans there
// (and a slack for the roundings), so no token at or past it shares a key with
// the bin.  Logits in [z0, z1) are listed; z0 lies below the bin's lower edge by
// as much, so the list holds the whole bin and every token that shares a key
// with it.
struct Bounds {
  float z0, z1;
};
template <bool VEC>
__device__ __forceinline__ Bounds bin_bounds(const Row<VEC>& row, int bin) {
  const double hi = (0.5 - bin) * (kLn2 / kOctave), lo = hi - kLn2 / kOctave;
  const double z1 = row.m + (hi + 2.0 / (exp(hi) * 0x1p40) + 1e-9) / row.inv_t;
  const double z0 = row.m + (lo - 2.0 / (exp(lo) * 0x1p40) - 1e-9) / row.inv_t;
  return {(float)(z0 - fabs(z0) * 0x1p-22), (float)(z1 + fabs(z1) * 0x1p-22)};
}
// Whether one key spans more than about a bin there (masses below kMinKey).
__device__ __forceinline__ bool bin_deep(int bin) {
  return exp(-(double)bin * (kLn2 / kOctave)) * 0x1p40 < kMinKey;
}

// A range of keys in kBins equal parts, the highest keys first.
struct Keys {
  uint64_t lo, hi;  // 1 <= lo <= hi
  int shift;        // a part is 2^shift keys
  __device__ __forceinline__ uint32_t part(uint64_t q) const { return (uint32_t)((hi - q) >> shift); }
  __device__ __forceinline__ bool has(uint64_t q) const { return q >= lo && q <= hi; }
};
__device__ __forceinline__ Keys make_keys(uint64_t lo, uint64_t hi) {
  static_assert(kBins == 1 << 10, "parts of the key range");
  return {lo, hi, max(0, 64 - __clzll((long long)(hi - lo) | 1) - 10)};
}
// The keys that tokens of a bin can have, with room for the roundings.
__device__ __forceinline__ Keys bin_keys(int bin) {
  const double hi = (0.5 - bin) * (kLn2 / kOctave), lo = hi - kLn2 / kOctave;
  const uint64_t k0 = scalar((uint64_t)(exp(lo) * (0x1p40 * (1.0 - 1e-9))));
  const uint64_t k1 = scalar((uint64_t)(exp(hi) * (0x1p40 * (1.0 + 1e-9))));
  return make_keys(k0 > 3 ? k0 - 2 : 1, k1 + 2);
}
// Whether the tokens of a bin of this total mass may be more than `cap` (a bound
// within 5% of their number), or too deep for the list's bounds.
__device__ __forceinline__ bool bin_wide(int bin, uint64_t mass, int cap) {
  return bin_deep(bin) || mass / bin_keys(bin).lo > (uint64_t)cap;
}

// Step 3 for a part of a slab at token `at`: the lane's mass of tokens at or above z1
// is returned, tokens of [z0, z1) go to the list (count in *n_list, which may
// pass cap; only the first cap are stored).
template <bool VEC>
__device__ __forceinline__ uint64_t slab_members(const Row<VEC>& row, const FastMass& fm, int at,
                                                 int part, const float (&v)[4], const Bounds& bd,
                                                 int lane, int cap, int* n_list, float* list_z,
                                                 int* list_i) {
  uint32_t mem = 0, lst = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    mem |= v[k] >= bd.z1 ? 1u << k : 0u;
    lst |= v[k] >= bd.z0 ? 1u << k : 0u;
  }
  lst &= ~mem;
  while (lst) {
    const int k = __ffs(lst) - 1, pos = atomicAdd(n_list, 1);
    lst &= lst - 1;
    if (pos < cap) {
      list_z[pos] = pick4(v, k);
      list_i[pos] = at + row.offset(part, k, lane);
    }
  }
  if (__any(__popc(mem) > 2)) {  // most of the slab
    float w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = mem >> k & 1 ? v[k] : -INFINITY;
    return slab_mass_all(row, fm, w);
  }
  return slab_mass(row, fm, v, mem);
}

// The passes over rows whose threshold bin is wide.

// Calls f(k, q) for the lane's tokens below z1.
template <bool VEC, typename F>
__device__ __forceinline__ void slab_below(const Row<VEC>& row, const FastMass& fm, const float (&v)[4],
                                           float z1, F&& f) {
  uint32_t mask = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) mask |= v[k] < z1 && v[k] > -INFINITY ? 1u << k : 0u;
  while (mask) {
    const int k = __ffs(mask) - 1;
    mask &= mask - 1;
    const float z[1] = {pick4(v, k)};
    uint64_t q[1];
    int bin[1];
    if (__builtin_expect(fast_mass<1>(fm, z, q, bin), 0)) q[0] = mass_at(row.x(z[0]));
    f(k, q[0]);
  }
}
// A logit at or above which every key is above `key`, with far more room than the
// float arithmetic needs (T above 10^36 only makes it higher than it has to be).
__device__ __forceinline__ float above_key(const FastMass& fm, uint64_t key) {
  const float x = (__builtin_amdgcn_logf((float)(key + 1)) - 40.f) * (float)kLn2 + 1e-4f;
  const float m = (float)fm.m, xt = x * fm.c.t;
  return scalar(m + xt + (fabsf(m) + fabsf(xt)) * 0x1p-20f + 1e-37f);
}

// Over blocks b0, b0 + step, .. below b1: the masses of bin `bin` whose keys lie in
// `keys`, by part, and every block's whole mass.
template <bool VEC>
__device__ __forceinline__ void sum_parts(const Row<VEC>& row, const FastMass& fm, int bin,
                                          const Keys& keys, int b0, int b1, int step,
                                          uint64_t* hist, uint64_t* bmass) {
  const int lane = threadIdx.x & 63;
  uint64_t total = 0;
  row.slabs(b0, b1, step, lane, [&](int b, int, int, const float(&v)[4], bool end) {
    uint64_t q[4];
    int bins[4];
    uint32_t redo = fast_mass<4>(fm, v, q, bins);
#pragma unroll 1
    for (; redo; redo &= redo - 1) {
      const int at = __ffs(redo) - 1;
      const uint64_t e = mass_at(row.x(pick4(v, at)));
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = k == at ? e : q[k];
    }
    uint32_t part[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      total += q[k];
      part[k] = keys.part(q[k]);
      q[k] = bins[k] == bin && keys.has(q[k]) ? q[k] : 0;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // runs of one part in a lane as one
      if (k < 3 && part[k] == part[k + 1]) q[k + 1] += q[k];
      else if (q[k]) atomicAdd((unsigned long long*)&hist[part[k]], q[k]);
    }
    if (end) {
      total = wave_sum_u64(total);
      if (lane == 0) bmass[b] = total;
      total = 0;
    }
  });
}

// LDS of the one-row work groups.
struct RowShared {
  uint64_t hist[kBins];
  uint64_t list_q[kListCap];
  float list_z[kListCap];
  int list_i[kListCap];
  uint64_t bmass[kMaxBlocks], bties[kMaxBlocks];
  uint64_t wave_s[kWaves];
  uint64_t small_q[64];
  double table[16];
  uint64_t sel_before, sel_total, kappa, kmin, kmax;
  float red_f[kWaves];
  int sel_rank, n_list, n_small, tie_cut;
};

// Thread t holds h, the mass of rank t.  Finds the first rank whose running
// mass from `above` reaches t_p (t_p > above); sel_rank = -1 if none does.
// sel_total is the sum of all ranks.
__device__ __forceinline__ void select_rank(RowShared& sh, uint64_t h, uint64_t above,
                                            uint64_t t_p) {
  const int t = thread_id(), lane = t & 63, wave = scalar(t >> 6);
  const uint64_t incl = wave_scan_incl(h);
  __syncthreads();
  if (lane == 63) sh.wave_s[wave] = incl;
  if (t == 0) sh.sel_rank = -1;
  __syncthreads();
  uint64_t before = above + incl - h, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) before += sh.wave_s[w];
    total += sh.wave_s[w];
  }
  if (before < t_p && before + h >= t_p) {
    sh.sel_rank = t;
    sh.sel_before = before;
  }
  if (t == 0) sh.sel_total = total;
  __syncthreads();
}

__device__ __forceinline__ uint64_t group_sum_u64(RowShared& sh, uint64_t v) {
  const int t = thread_id();
  v = wave_sum_u64(v);
  __syncthreads();
  if ((t & 63) == 0) sh.wave_s[t >> 6] = v;
  __syncthreads();
  uint64_t total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) total += sh.wave_s[w];
  return scalar(total);
}

// What the last steps need to know of the nucleus: its keys are q > kappa,
// and q == kappa up to token tie_cut.
struct Nucleus {
  uint64_t kappa;
  int tie_cut;
};

// The largest key of the n listed ones whose mass from `above` reaches t_p, by radix
// select: digits of 10 bits, five rounds.
__device__ uint64_t radix_key(RowShared& sh, int n, uint64_t above, uint64_t t_p) {
  uint64_t prefix = 0;
#pragma unroll 1
  for (int r = 0; r < 5; ++r) {
    const int t = thread_id();
    const int shift = r < 4 ? 31 - 10 * r : 0, width = r < 4 ? 10 : 1;  // bits 40..31, .., 10..1, 0
    __syncthreads();
    sh.hist[t] = zero_u64();
    __syncthreads();
    for (int e = t; e < n; e += kThreads) {
      const uint64_t q = sh.list_q[e];
      if (q != 0 && (q >> (shift + width)) == prefix)
        atomicAdd((unsigned long long*)&sh.hist[(q >> shift) & ((1u << width) - 1)], q);
    }
    __syncthreads();
    const int bins = 1 << width, rank = t;
    select_rank(sh, rank < bins ? sh.hist[bins - 1 - rank] : 0, above, t_p);
    prefix = (prefix << width) | (uint64_t)(bins - 1 - scalar(sh.sel_rank));
    above = scalar(sh.sel_before);
  }
  return prefix;
}

// Walks tokens [at, at + n) in index order with weight w(token, q); returns
// the first token whose running weight from `before` reaches `need`, or -1.
template <bool VEC, typename W>
__device__ int walk(RowShared& sh, const Row<VEC>& row, int at, int n, uint64_t before, uint64_t need,
                    W&& w) {
  for (int o = 0; o < n; o += kThreads) {
    const int i = at + o + threadIdx.x;
    uint64_t h = 0;
    if (o + (int)threadIdx.x < n) h = w(i, mass_at(row.x(row.z[i])));
    select_rank(sh, h, before, need);
    const int found = scalar(sh.sel_rank);
    before += scalar(sh.sel_total);
    if (found >= 0) return at + o + found;
  }
  return -1;
}

// The index of the n_tie-th token with key kappa, in index order (bties holds the
// blocks' numbers of them), and the block it lies in.
template <bool VEC>
__device__ int last_tie(RowShared& sh, const Row<VEC>& row, uint64_t kappa, uint64_t n_tie, int& block,
                        uint64_t& before) {
  const int t = thread_id();
  select_rank(sh, t < row.nb ? sh.bties[t] : 0, 0, n_tie);
  block = max(scalar(sh.sel_rank), 0);
  before = scalar(sh.sel_before);
  const int at = block * row.blen;
  return walk(sh, row, at, min(row.blen, row.V - at), before, n_tie,
              [&](int, uint64_t q) -> uint64_t { return q == kappa; });
}

// Ties and the blocks' nucleus masses from kappa alone (bmass: the blocks' whole
// masses), by a pass over the tokens at kappa and below; false if the key is not kappa.
template <bool VEC>
__device__ bool key_threshold(RowShared& sh, const Row<VEC>& row, const FastMass& fm, uint64_t kappa,
                              uint64_t t_p, Nucleus& nu) {
  const int t = thread_id(), lane = t & 63, wave = scalar(t >> 6);
  const float z1 = above_key(fm, kappa);
  uint64_t below = 0, ties = 0;
  row.slabs(wave, row.nb, kWaves, lane, [&](int b, int, int, const float(&v)[4], bool end) {
    slab_below(row, fm, v, z1, [&](int, uint64_t q) {
      below += q <= kappa ? q : 0;
      ties += q == kappa;
    });
    if (end) {
      below = wave_sum_u64(below);
      ties = wave_sum_u64(ties);
      if (lane == 0) {
        sh.bmass[b] -= below;
        sh.bties[b] = ties;
      }
      below = ties = 0;
    }
  });
  __syncthreads();
  const uint64_t above = group_sum_u64(sh, t < row.nb ? sh.bmass[t] : 0);
  const uint64_t n_all = group_sum_u64(sh, t < row.nb ? sh.bties[t] : 0);
  if (above >= t_p || above + n_all * kappa < t_p) return false;
  const uint64_t n_tie = (t_p - above + kappa - 1) / kappa;
  int tb;
  uint64_t tie0;
  const int cut = last_tie(sh, row, kappa, n_tie, tb, tie0);
  if (t < row.nb) {
    const uint64_t members = t < tb ? sh.bties[t] : t == tb ? n_tie - tie0 : 0;
    sh.bmass[t] += members * kappa;
  }
  __syncthreads();
  nu = {kappa, cut};
  return true;
}

// Step 4: kappa, ties and the blocks' nucleus masses from the list: n tokens, every
// token with a key in `keys` among them (a few outside it count at its ends); bmass
// holds the masses above the list.
template <bool VEC>
__device__ Nucleus list_threshold(RowShared& sh, const Row<VEC>& row, const Keys& keys, int n,
                                  uint64_t t_p) {
  const int t = thread_id(), lane = t & 63, wave = scalar(t >> 6);
  const uint64_t above1 = group_sum_u64(sh, t < row.nb ? sh.bmass[t] : 0);
  auto part = [&](uint64_t q) { return q >= keys.hi ? 0 : min((uint32_t)kBins - 1, keys.part(max(q, keys.lo))); };
  sh.hist[t] = zero_u64();
  if (t == 0) {
    sh.n_small = 0;
    sh.kmin = ~0ull;
    sh.kmax = 0;
  }
  __syncthreads();
  for (int e = t; e < n; e += kThreads) {
    const uint64_t q = mass_at(row.x(sh.list_z[e]));
    sh.list_q[e] = q;
    if (q) atomicAdd((unsigned long long*)&sh.hist[part(q)], q);
  }
  __syncthreads();
  select_rank(sh, sh.hist[t], above1, t_p);
  const uint32_t sub = scalar(sh.sel_rank);
  const uint64_t above_s = scalar(sh.sel_before);
  for (int e = t; e < n; e += kThreads) {
    const uint64_t q = sh.list_q[e];
    if (q && part(q) == sub) {
      const int p = atomicAdd(&sh.n_small, 1);
      if (p < 64) sh.small_q[p] = q;
    }
  }
  __syncthreads();
  const int ns = scalar(sh.n_small);
  uint64_t kappa;
  if (ns <= 64) {
    if (wave == 0) {
      const uint64_t q = lane < ns ? sh.small_q[lane] : 0;
      uint64_t gt = above_s, eq = 0;
      for (int j = 0; j < ns; ++j) {
        const uint64_t o = lane_u64(q, j);
        gt += o > q ? o : 0;
        eq += o == q ? o : 0;
      }
      if (q && gt < t_p && gt + eq >= t_p) sh.kappa = q;
    }
    __syncthreads();
    kappa = scalar(sh.kappa);
  } else {  // many tokens in one part: mostly one key (coarsely rounded logits)
    uint64_t lo = ~0ull, hi = 0;
    for (int e = t; e < n; e += kThreads) {
      const uint64_t q = sh.list_q[e];
      if (!q || part(q) != sub) continue;
      lo = min(lo, q);
      hi = max(hi, q);
    }
    if (hi) {
      atomicMin((unsigned long long*)&sh.kmin, lo);
      atomicMax((unsigned long long*)&sh.kmax, hi);
    }
    __syncthreads();
    kappa = scalar(sh.kmin);
    if (kappa != scalar(sh.kmax)) kappa = radix_key(sh, n, above1, t_p);
  }
  uint64_t strict = 0, ties = 0;
  for (int e = t; e < n; e += kThreads) {
    const uint64_t q = sh.list_q[e];
    strict += q > kappa ? q : 0;
    ties += q == kappa;
  }
  const uint64_t above = above1 + group_sum_u64(sh, strict);
  ties = group_sum_u64(sh, ties);
  const uint64_t n_tie = (t_p - above + kappa - 1) / kappa;
  int cut = INT_MAX;
  if (n_tie < ties) {  // ties join in index order: the last member's index
    if (t < row.nb) sh.bties[t] = zero_u64();
    __syncthreads();
    for (int e = t; e < n; e += kThreads)
      if (sh.list_q[e] == kappa)
        atomicAdd((unsigned long long*)&sh.bties[sh.list_i[e] / row.blen], 1ull);
    __syncthreads();
    int tb;
    uint64_t tie0;
    cut = last_tie(sh, row, kappa, n_tie, tb, tie0);
  }
  for (int e = t; e < n; e += kThreads) {
    const uint64_t q = sh.list_q[e];
    if (q > kappa || (q == kappa && sh.list_i[e] <= cut))
      atomicAdd((unsigned long long*)&sh.bmass[sh.list_i[e] / row.blen], q);
  }
  __syncthreads();
  return {kappa, cut};
}

// Step 3 for a row whose threshold bin has too many tokens to list, or keys so low
// that one spans several bins.  The bin's keys are cut into kBins parts and the part
// that crosses t_p found, as step 2 does with the bins (`counted`: hist and bmass are
// there already).  Where its tokens fit they are listed, `keys` is the part, and 0 is
// returned; where a sample of them has one key, that is (many logits are equal, and
// key_threshold says whether it is kappa); otherwise the part is cut again.  `above` is
// the mass of the bins above this one.  Only the bin's own tokens are counted: those
// of higher bins have its keys or higher ones, so kappa is the same.
template <bool VEC>
__device__ uint64_t cut_bin(RowShared& sh, const Row<VEC>& row, const FastMass& fm, int bin,
                            uint64_t& above, uint64_t t_p, bool& counted, Keys& keys) {
  for (;;) {
    const int t = thread_id(), lane = t & 63, wave = scalar(t >> 6);
    if (!counted) {
      __syncthreads();
      sh.hist[t] = zero_u64();
      __syncthreads();
      sum_parts(row, fm, bin, keys, wave, row.nb, kWaves, sh.hist, sh.bmass);
      __syncthreads();
    }
    counted = false;
    select_rank(sh, sh.hist[t], above, t_p);
    const uint64_t rank = scalar(sh.sel_rank), mass = scalar(sh.hist[rank]);
    above = scalar(sh.sel_before);
    const uint64_t top = keys.hi - (rank << keys.shift);
    if (keys.shift == 0) return top;
    const uint64_t width = (1ull << keys.shift) - 1;
    keys = make_keys(top > keys.lo + width ? top - width : keys.lo, top);
    if (t == 0) {
      sh.n_list = sh.n_small = 0;
      sh.kmin = ~0ull;
      sh.kmax = 0;
    }
    __syncthreads();
    // Tokens of the part, within 0.1%: distinct logits leave it V / 1000 or so, more of
    // them are mostly equal, which a sample (the row's first tokens) shows.
    const uint64_t count = mass / keys.lo;
    if (count > kThreads) {
      const uint64_t q = t < row.V ? mass_at(row.x(row.z[t])) : 0;
      if (keys.has(q)) {
        atomicMin((unsigned long long*)&sh.kmin, q);
        atomicMax((unsigned long long*)&sh.kmax, q);
        atomicAdd(&sh.n_small, 1);
      }
      __syncthreads();
      const uint64_t one = scalar(sh.kmin);
      if (scalar(sh.n_small) >= 4 && one == scalar(sh.kmax)) return one;
    }
    if (count > kListCap) continue;
    const float z1 = above_key(fm, keys.hi);
    uint64_t below = 0;
    row.slabs(wave, row.nb, kWaves, lane, [&](int b, int at, int part, const float(&v)[4], bool end) {
      slab_below(row, fm, v, z1, [&](int k, uint64_t q) {
        if (q > keys.hi) return;
        below += q;
        if (q < keys.lo) return;
        const int pos = atomicAdd(&sh.n_list, 1);
        if (pos >= kListCap) return;
        sh.list_z[pos] = pick4(v, k);
        sh.list_i[pos] = at + row.offset(part, k, lane);
      });
      if (end) {
        below = wave_sum_u64(below);
        if (lane == 0) sh.bmass[b] -= below;
        below = 0;
      }
    });
    __syncthreads();
    if (sh.n_list <= kListCap) return 0;
  }
}

// Step 4, after step 3 (the bin's tokens are listed) or with it.
template <bool VEC>
__device__ __forceinline__ Nucleus threshold(RowShared& sh, const Row<VEC>& row, const FastMass& fm,
                                             int bin, uint64_t above, uint64_t t_p, bool listed,
                                             bool counted) {
  Keys keys = bin_keys(bin);
  Nucleus nu{0, INT_MAX};
  // A range of under 2^36 keys is down to single ones after four cuts.
  for (int round = 0; round < 6; ++round) {
    const uint64_t key = listed ? 0 : cut_bin(sh, row, fm, bin, above, t_p, counted, keys);
    if (key == 0) return list_threshold(sh, row, keys, scalar(sh.n_list), t_p);
    if (key_threshold(sh, row, fm, key, t_p, nu)) break;
  }
  return nu;
}

// Step 5: the block that holds the target, then its token.
template <bool VEC>
__device__ void take_token(RowShared& sh, const Row<VEC>& row, const Nucleus& nu, float u,
                           int32_t* token) {
  const int t = thread_id();
  const uint64_t Z = group_sum_u64(sh, t < row.nb ? sh.bmass[t] : 0);
  u = fminf(fmaxf(u, 0.f), 0x1.fffffep-1f);
  const uint64_t u24 = (uint64_t)(u * 0x1p24f);
  const uint64_t target = (uint64_t)(((u128)u24 * Z) >> 24);
  select_rank(sh, t < row.nb ? sh.bmass[t] : 0, 0, target + 1);
  const int b = scalar(sh.sel_rank);
  if (b < 0) return;  // no mass at all (a row without finite logits): no token
  const uint64_t before = scalar(sh.sel_before);
  const int at = b * row.blen;
  const int i = walk(sh, row, at, min(row.blen, row.V - at), before, target + 1,
                     [&](int tok, uint64_t q) -> uint64_t {
                       return q > nu.kappa || (q == nu.kappa && tok <= nu.tie_cut) ? q : 0;
                     });
  if (t == 0 && i >= 0) *token = i;
}

__device__ __forceinline__ uint64_t threshold_mass(uint32_t p24, uint64_t S) {
  return (uint64_t)(((u128)p24 * S + ((u128)1 << 24) - 1) >> 24);
}

// Steps 2 to 5 of one row by one work group of kThreads.
template <bool VEC>
__device__ void sample_row(RowShared& sh, const Row<VEC>& row, const Scale& sc, uint32_t p24, float u,
                           int32_t* token) {
  const int t = threadIdx.x, lane = t & 63, wave = scalar(t >> 6);
  const FastMass fm = make_fast(row.m, sc, sh.table);
  fill_table(sh.table);
  if (t == 0) sh.n_list = 0;
  sh.hist[t] = zero_u64();
  __syncthreads();
  uint64_t sum = 0;
  auto end_block = [&](int b) {
    sum = wave_sum_u64(sum);
    if (lane == 0) sh.bmass[b] = sum;
    sum = 0;
  };
  if (p24 == 1u << 24) {  // every token of nonzero mass
    row.slabs(wave, row.nb, kWaves, lane, [&](int b, int, int, const float(&v)[4], bool end) {
      sum += slab_mass_all(row, fm, v);
      if (end) end_block(b);
    });
    __syncthreads();
    take_token(sh, row, {0, INT_MAX}, u, token);
    return;
  }
  row.slabs(wave, row.nb, kWaves, lane,
            [&](int, int, int, const float(&v)[4], bool) { slab_hist(row, fm, v, sh.hist); });
  __syncthreads();
  const uint64_t S = group_sum_u64(sh, sh.hist[t]);
  if (S == 0) return;  // a row without finite logits
  const uint64_t t_p = scalar(threshold_mass(p24, S));
  select_rank(sh, sh.hist[t], 0, t_p);
  const int bin = scalar(sh.sel_rank);
  const uint64_t above = scalar(sh.sel_before);
  bool listed = !bin_wide(bin, sh.hist[bin], kListCap);
  if (listed) {
    const Bounds bd = bin_bounds(row, bin);
    row.slabs(wave, row.nb, kWaves, lane, [&](int b, int at, int part, const float(&v)[4], bool end) {
      sum += slab_members(row, fm, at, part, v, bd, lane, kListCap, &sh.n_list, sh.list_z, sh.list_i);
      if (end) end_block(b);
    });
    __syncthreads();
    listed = sh.n_list <= kListCap;
  }
  const Nucleus nu = threshold(sh, row, fm, bin, above, t_p, listed, false);
  take_token(sh, row, nu, u, token);
}

// Row maximum by a work group of kThreads: eight 16-byte loads in flight per lane.
template <bool VEC>
__device__ float row_max_group(RowShared& sh, const Row<VEC>& row) {
  const int t = threadIdx.x;
  float mx = -INFINITY;
  if constexpr (VEC) {
    const int n4 = row.V / 4;
    for (int base = 0; base < n4; base += 8 * kThreads) {
      float4 f[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) f[u] = ((const float4*)row.z)[min(base + u * kThreads + t, n4 - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        mx = fmaxf(mx, fmaxf(fmaxf(f[u].x, f[u].y), fmaxf(f[u].z, f[u].w)));
    }
  } else {
    for (int64_t base = 0; base < row.V; base += 8 * kThreads) {
      float f[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        f[u] = row.z[min(base + u * kThreads + t, (int64_t)row.V - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) mx = fmaxf(mx, f[u]);
    }
  }
  mx = wave_max(mx);
  if ((t & 63) == 0) sh.red_f[t >> 6] = mx;
  __syncthreads();
  mx = sh.red_f[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, sh.red_f[w]);
  return mx;
}

template <bool VEC>
__global__ __launch_bounds__(kThreads) void sample_top_p_kernel(
    int V, const float* __restrict__ logits, Scale sc, uint32_t p24,
    const float* __restrict__ uniforms, int32_t* __restrict__ tokens) {
  __shared__ RowShared sh;
  const int b = blockIdx.x;
  Row<VEC> row = make_row<VEC>(V, logits, b, sc);
  row.m = scalar((double)row_max_group(sh, row));
  sample_row(sh, row, sc, p24, uniforms[b], tokens + b);
}

// ---------------------------------------------------------------------------
// Split form for small batches.  One work group per row leaves most CUs idle
// and each pass over a 513 KB row runs at one CU's rate; here the three passes
// over the row are spread over C work groups per row, each owning a run of the
// row's index blocks, and steps 2's decision and 4 to 5 run on one group per
// row between and after them:
//   split_max -> split_hist -> split_bin -> split_members -> split_finish
// (without the histogram and its decision when top_p = 1).  All cross-chunk
// results are integer sums, maxima and an unordered list, so the token is the
// one-group form's.
// ---------------------------------------------------------------------------
constexpr int kST = 512, kSW = kST / 64;  // threads / waves of the chunk kernels

struct RowState {
  uint64_t t_p, above;  // above: the mass of the bins above the threshold bin
  int32_t bin;          // threshold bin; -1: no mass in the row
  int32_t wide;         // the bin is cut into parts (wide_threshold), not listed
};

struct SplitWs {
  RowState* st;    // [B]
  float* cmax;     // [B][C]
  uint64_t* hist;  // [B][C][kBins], by bin, then by part of a wide bin
  uint64_t* bmass; // [B][kMaxBlocks]
  int* count;      // [B][C] listed tokens of a chunk (may pass cap)
  float* list_z;   // [B][C][cap]
  int* list_i;     // [B][C][cap]
  int C, cap;
};

// Blocks of chunk c: [b0, b1).
__device__ __forceinline__ void chunk_blocks(int nb, int C, int c, int& b0, int& b1) {
  const int per = (nb + C - 1) / C;
  b0 = min(nb, c * per);
  b1 = min(nb, b0 + per);
}

// Row max from the chunk maxima (the same float max as one pass); C <= 64.
__device__ __forceinline__ double split_row_max(const SplitWs& ws, int b) {
  const int lane = threadIdx.x & 63;
  const float v = lane < ws.C ? ws.cmax[(int64_t)b * ws.C + lane] : -INFINITY;
  return scalar((double)wave_max(v));
}

template <bool VEC>
__global__ __launch_bounds__(kST) void split_max(int V, const float* __restrict__ logits,
                                                 SplitWs ws) {
  __shared__ float red[kSW];
  const int c = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, wave = scalar((int)threadIdx.x >> 6);
  const Row<VEC> row = make_row<VEC>(V, logits, b, Scale{});
  int b0, b1;
  chunk_blocks(row.nb, ws.C, c, b0, b1);
  float mx = -INFINITY;
  row.slabs(b0 + wave, b1, kSW, lane, [&](int, int, int, const float(&v)[4], bool) {
#pragma unroll
    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, v[i]);
  });
  mx = wave_max(mx);
  if (lane == 0) red[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kSW; ++w) mx = fmaxf(mx, red[w]);
    ws.cmax[(int64_t)b * ws.C + c] = mx;
  }
}

template <bool VEC>
__global__ __launch_bounds__(kST) void split_hist(int V, const float* __restrict__ logits,
                                                  Scale sc, SplitWs ws) {
  __shared__ uint64_t hist[kBins];
  __shared__ double table[16];
  const int c = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, wave = scalar((int)threadIdx.x >> 6);
  Row<VEC> row = make_row<VEC>(V, logits, b, sc);
  row.m = split_row_max(ws, b);
  const FastMass fm = make_fast(row.m, sc, table);
  fill_table(table);
  for (int i = threadIdx.x; i < kBins; i += kST) hist[i] = 0;
  __syncthreads();
  int b0, b1;
  chunk_blocks(row.nb, ws.C, c, b0, b1);
  row.slabs(b0 + wave, b1, kSW, lane,
            [&](int, int, int, const float(&v)[4], bool) { slab_hist(row, fm, v, hist); });
  __syncthreads();
  uint64_t* dst = ws.hist + ((int64_t)b * ws.C + c) * kBins;
  for (int i = threadIdx.x; i < kBins; i += kST) dst[i] = hist[i];
}

// Entry threadIdx.x of the row's histogram, over its chunks.
__device__ __forceinline__ uint64_t chunk_hists(const SplitWs& ws, int b) {
  const uint64_t* h0 = ws.hist + (int64_t)b * ws.C * kBins + threadIdx.x;
  uint64_t h = 0;
  for (int c0 = 0; c0 < ws.C; c0 += 8) {  // C is a multiple of 8
    uint64_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = h0[(int64_t)(c0 + u) * kBins];
#pragma unroll
    for (int u = 0; u < 8; ++u) h += v[u];
  }
  return h;
}

__global__ __launch_bounds__(kThreads) void split_bin(uint32_t p24, SplitWs ws) {
  __shared__ RowShared sh;
  const int b = blockIdx.x, t = threadIdx.x;
  const uint64_t h = chunk_hists(ws, b);
  const uint64_t S = group_sum_u64(sh, h);
  RowState st{0, 0, -1, 0};
  if (S != 0) {
    st.t_p = threshold_mass(p24, S);
    sh.hist[t] = h;
    select_rank(sh, h, 0, st.t_p);
    st.bin = sh.sel_rank;
    st.above = sh.sel_before;
    // A quarter of the chunks' lists for their unequal shares.
    st.wide = bin_wide(st.bin, sh.hist[st.bin], min(kListCap, ws.C * ws.cap / 4 * 3));
  }
  if (t == 0) ws.st[b] = st;
}

template <bool VEC>
__global__ __launch_bounds__(kST) void split_members(int V, const float* __restrict__ logits,
                                                     Scale sc, int all, SplitWs ws) {
  __shared__ int n_list;
  __shared__ double table[16];
  __shared__ uint64_t hist[kBins];
  const int c = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, wave = scalar((int)threadIdx.x >> 6);
  Row<VEC> row = make_row<VEC>(V, logits, b, sc);
  row.m = split_row_max(ws, b);
  int b0, b1;
  chunk_blocks(row.nb, ws.C, c, b0, b1);
  uint64_t* bmass = ws.bmass + (int64_t)b * kMaxBlocks;
  const FastMass fm = make_fast(row.m, sc, table);
  fill_table(table);
  if (threadIdx.x == 0) n_list = 0;
  __syncthreads();
  uint64_t sum = 0;
  auto end_block = [&](int k) {
    sum = wave_sum_u64(sum);
    if (lane == 0) bmass[k] = sum;
    sum = 0;
  };
  if (all) {  // top_p = 1
    row.slabs(b0 + wave, b1, kSW, lane, [&](int k, int, int, const float(&v)[4], bool end) {
      sum += slab_mass_all(row, fm, v);
      if (end) end_block(k);
    });
    return;
  }
  RowState st = ws.st[b];
  st.bin = scalar(st.bin);
  if (st.bin < 0) return;  // uniform over the group
  if (st.wide) {
    for (int i = threadIdx.x; i < kBins; i += kST) hist[i] = 0;
    __syncthreads();
    sum_parts(row, fm, st.bin, bin_keys(st.bin), b0 + wave, b1, kSW, hist, bmass);
    __syncthreads();
    uint64_t* dst = ws.hist + ((int64_t)b * ws.C + c) * kBins;
    for (int i = threadIdx.x; i < kBins; i += kST) dst[i] = hist[i];
    return;
  }
  const Bounds bd = bin_bounds(row, st.bin);
  const int64_t at0 = ((int64_t)b * ws.C + c) * ws.cap;
  row.slabs(b0 + wave, b1, kSW, lane, [&](int k, int at, int part, const float(&v)[4], bool end) {
    sum += slab_members(row, fm, at, part, v, bd, lane, ws.cap, &n_list, ws.list_z + at0,
                        ws.list_i + at0);
    if (end) end_block(k);
  });
  __syncthreads();
  if (threadIdx.x == 0) ws.count[(int64_t)b * ws.C + c] = n_list;
}

template <bool VEC>
__global__ __launch_bounds__(kThreads) void split_finish(int V, const float* __restrict__ logits,
                                                         Scale sc, int all,
                                                         const float* __restrict__ uniforms,
                                                         int32_t* __restrict__ tokens, SplitWs ws) {
  __shared__ RowShared sh;
  __shared__ int base[65];
  const int b = blockIdx.x, t = threadIdx.x;
  Row<VEC> row = make_row<VEC>(V, logits, b, sc);
  row.m = split_row_max(ws, b);
  Nucleus nu{0, INT_MAX};
  if (all) {
    if (t < row.nb) sh.bmass[t] = ws.bmass[(int64_t)b * kMaxBlocks + t];
    __syncthreads();
  } else {
    RowState st = ws.st[b];
    st.t_p = scalar(st.t_p);
    st.above = scalar(st.above);
    st.bin = scalar(st.bin);
    if (st.bin < 0) return;  // a row without finite logits
    const FastMass fm = make_fast(row.m, sc, sh.table);
    bool listed = !st.wide;
    if (listed) {
      if (t == 0) {  // where each chunk's tokens start in the row's list
        int n = 0;
        bool fits = true;
        for (int c = 0; c < ws.C; ++c) {
          base[c] = n;
          const int k = ws.count[(int64_t)b * ws.C + c];
          fits = fits && k <= ws.cap;
          n += min(k, ws.cap);
        }
        base[ws.C] = n;
        sh.n_list = fits && n <= kListCap ? n : -1;
      }
      if (t < row.nb) sh.bmass[t] = ws.bmass[(int64_t)b * kMaxBlocks + t];
      __syncthreads();
      listed = sh.n_list >= 0;
    }
    if (listed) {
      for (int c = t >> 6; c < ws.C; c += kWaves) {
        const int64_t at0 = ((int64_t)b * ws.C + c) * ws.cap;
        for (int e = t & 63; e < base[c + 1] - base[c]; e += 64) {
          sh.list_z[base[c] + e] = ws.list_z[at0 + e];
          sh.list_i[base[c] + e] = ws.list_i[at0 + e];
        }
      }
      __syncthreads();
    } else {
      fill_table(sh.table);
      if (st.wide) {  // counted by split_members
        sh.hist[t] = chunk_hists(ws, b);
        if (t < row.nb) sh.bmass[t] = ws.bmass[(int64_t)b * kMaxBlocks + t];
      }
      __syncthreads();
    }
    nu = threshold(sh, row, fm, st.bin, st.above, st.t_p, listed, st.wide);
  }
  take_token(sh, row, nu, uniforms[b], tokens + b);
}

}  // namespace

namespace {

// Chunks per row: about 256 work groups per pass.  Above 32 rows one group per
// row: the split form would need scratch that grows with the batch, and its
// callers hold none there.
constexpr int sample_split_chunks(int B) { return B <= 8 ? 32 : B <= 16 ? 16 : B <= 32 ? 8 : 1; }
// Listed tokens a chunk may hold: twice its share of a full list (its share above 16
// rows), so that only rows whose tokens of one bin stand close together pass it.
constexpr int sample_list_cap(int C) { return C == 32 ? 512 : 1024; }

constexpr int64_t al256(int64_t x) { return (x + 255) & ~(int64_t)255; }

constexpr int64_t split_workspace_bytes(int B) {
  const int C = sample_split_chunks(B);
  return C == 1 ? 0
                : al256((int64_t)B * sizeof(RowState)) + al256((int64_t)B * C * 4) +
                      al256((int64_t)B * C * kBins * 8) + al256((int64_t)B * kMaxBlocks * 8) +
                      al256((int64_t)B * C * 4) + 2 * al256((int64_t)B * C * sample_list_cap(C) * 4) +
                      256;
}

constexpr int64_t max_split_workspace_bytes() {
  int64_t m = 0;
  for (int B = 1; B <= 256; ++B) m = split_workspace_bytes(B) > m ? split_workspace_bytes(B) : m;
  return m;
}

// ---------------------------------------------------------------------------
// Scratch of the no-allocation entry point (sample_top_p_noalloc): the split
// form's row states and per-chunk partial results in a static device array
// sized for the largest batch that takes the split form (about 4 MiB).  Each
// GPU the library runs on holds its own copy until the process ends; every
// call on a GPU shares that GPU's copy, so such calls must not overlap.  No
// entry of it needs clearing: every kernel of the split form writes what
// the next one reads before it is read.
// ---------------------------------------------------------------------------
constexpr int64_t kSampleScratchBytes = max_split_workspace_bytes();
__device__ __align__(256) char sample_scratch[kSampleScratchBytes];

std::mutex g_scratch_mu;
constexpr int kMaxDevices = 64;
void* g_scratch_dev[kMaxDevices] = {};

}  // namespace

int64_t sample_workspace_bytes(int B) { return split_workspace_bytes(B); }

int64_t sample_scratch_bytes() { return kSampleScratchBytes; }

// The device address of this GPU's copy of the scratch array.  In host code
// the array's name is only a host-side stand-in, so the address is looked up
// once per device (with that device current) and kept.
hipError_t sample_scratch_ptr(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(sample_scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return hipSuccess;
}

namespace {

template <bool VEC>
void launch_split(int B, int V, const float* logits, const Scale& scale, uint32_t p24,
                  const float* uniforms, int32_t* tokens, const SplitWs& ws, hipStream_t stream) {
  const dim3 grid(ws.C, B);
  const int all = p24 == 1u << 24;
  split_max<VEC><<<grid, kST, 0, stream>>>(V, logits, ws);
  if (!all) {
    split_hist<VEC><<<grid, kST, 0, stream>>>(V, logits, scale, ws);
    split_bin<<<B, kThreads, 0, stream>>>(p24, ws);
  }
  split_members<VEC><<<grid, kST, 0, stream>>>(V, logits, scale, all, ws);
  split_finish<VEC><<<B, kThreads, 0, stream>>>(V, logits, scale, all, uniforms, tokens, ws);
}

}  // namespace

hipError_t launch_sample_top_p(int B, int V, const float* logits, float temperature, float top_p,
                               const float* uniforms, int32_t* tokens, void* workspace,
                               int64_t ws_bytes, hipStream_t stream) {
  if (B == 0) return hipSuccess;
  const double inv_t = 1.0 / (double)temperature;
  const Scale scale{inv_t, -29.0 / inv_t, inv_t * (kOctave / kLn2), std::min(temperature, 1e36f)};
  uint32_t p24 = (uint32_t)rint((double)top_p * 16777216.0);
  p24 = p24 < 1 ? 1 : (p24 > (1u << 24) ? (1u << 24) : p24);
  // 16-byte loads need every row 16-byte aligned.
  const bool vec = (V & 3) == 0 && ((uintptr_t)logits & 15) == 0;
  const int C = sample_split_chunks(B);
  if (C == 1 || !workspace || ws_bytes < sample_workspace_bytes(B)) {
    if (vec)
      sample_top_p_kernel<true><<<B, kThreads, 0, stream>>>(V, logits, scale, p24, uniforms, tokens);
    else
      sample_top_p_kernel<false><<<B, kThreads, 0, stream>>>(V, logits, scale, p24, uniforms, tokens);
    return hipGetLastError();
  }
  // Workspace layout (256-byte aligned pieces, from an aligned start).
  char* p = (char*)(((uintptr_t)workspace + 255) & ~(uintptr_t)255);
  auto take = [&](int64_t bytes) {
    char* at = p;
    p += al256(bytes);
    return at;
  };
  SplitWs ws;
  ws.C = C;
  ws.cap = sample_list_cap(C);
  ws.st = (RowState*)take((int64_t)B * sizeof(RowState));
  ws.cmax = (float*)take((int64_t)B * C * 4);
  ws.hist = (uint64_t*)take((int64_t)B * C * kBins * 8);
  ws.bmass = (uint64_t*)take((int64_t)B * kMaxBlocks * 8);
  ws.count = (int*)take((int64_t)B * C * 4);
  ws.list_z = (float*)take((int64_t)B * C * ws.cap * 4);
  ws.list_i = (int*)take((int64_t)B * C * ws.cap * 4);
  if (vec)
    launch_split<true>(B, V, logits, scale, p24, uniforms, tokens, ws, stream);
  else
    launch_split<false>(B, V, logits, scale, p24, uniforms, tokens, ws, stream);
  return hipGetLastError();
}

}  // namespace pdec
