// pp_reduce.hip -- reduced exact solve of one worker's rooted-tree knapsack.
//
// k_reduce solves Eq. 9 for a chain without sweeping all n rows.  For a price
// lambda >= 0 let V(b) = p_b - lambda + sum over children c of max(V(c), 0),
// and S the nodes whose V and whose ancestors' V are all positive.  S
// maximises sum (p - lambda), so for every feasible set X
//     value(X) <= UB = lambda k' + sum over roots of max(V, 0),
// and X falls short of UB by at least
//     -V(a) for any ancestor-or-self a with V(a) < 0 of a node X takes,
//      V(a) for any ancestor-or-self a in S of a node of S that X leaves out.
// With a feasible set of value LB in hand and gap = UB - LB, every optimal
// set therefore leaves out each node below (or at) some V < -gap, and takes
// each node of S whose whole ancestor path has V > gap.  What is left, the
// core, is small (the gap is about the price of a fraction of one chunk: 64
// to 128 core nodes at n = 50,000, k = 4096).  LB comes from solving a core
// of guessed width D with the plain DP; the result stands if gap <= D, and
// otherwise the core of width D = gap is solved, which proves itself.
//
// The returned set is the full DP's, ties included.  The full DP's walk
// yields one particular optimal set X*, and every optimal set avoids the
// nodes left out and holds the forced ones.  On the rows the walk visits the
// reduced table holds the full table's values (X*'s suffix is feasible in
// the reduced problem, which only has fewer sets), a take row's skip value
// only shrinks and a skip row's take value only shrinks, so the reduced walk
// branches the same way everywhere.  For real-valued costs the same argument
// holds for the rounded values: rounding is monotone, so the full table's
// entries are the maxima of the sets' rounded sums; forced rows are kept in
// the reduced recurrence (D = p + D) so that every sum is rounded as there,
// and the gap includes the bound (1 + 2^-53)^k' on rounded sums.
//
// V is computed on integers: the profits themselves if their sum is below
// 2^47, else shifted right (integer costs) or scaled by a power of two and
// truncated (real-valued costs); truncation loses less than one unit per
// node, so UB is raised by k' units then.
//
// k_ladder first finds, for a ladder of prices t, a superset of S_t over the
// whole tree, one block per chain and price; k_reduce (one block of 1024
// threads per chain) takes the highest price whose set clearly exceeds k'.
// For a price lambda >= t, S is inside S_t, and any node outside S_t has an
// ancestor-or-self with V <= t - lambda, so it stays out as long as gap <
// lambda - t.  A chain that does not fit (too many active nodes, too wide a
// core) is left to the full sweep.
//
// Both kernels read the tree in level order (DevState::lvpos): internal
// nodes level by level from the roots, then every leaf.  Child sums live in
// LDS; leaves add theirs in one pass, internal nodes level by level with one
// barrier each.  Counters at n = 50,000, m = 16, k = 4,096 (shares of the
// waves' time, four waves a SIMD): k_ladder waits 70% (loads, LDS atomics,
// barriers) and issues 21%, so a SIMD issues most of the time and its vector
// unit is in use 40%; k_reduce waits 70% and issues 16%, vector 26%.  Loops
// that run once per launch are kept rolled (an unrolled ladder was slower).

#include <algorithm>

#include "pp_internal.h"

namespace pp {

namespace {

constexpr int kRThreads = kReduceThreads;
constexpr int kRWaves = kRThreads / 64;
// V words: V in the upper bits, the size of the subtree's part of S below
constexpr int kSizeBits = 14;
static_assert(kReduceActive < (1 << kSizeBits), "size field");
constexpr int kValueBits = 47;  // bound on the sum of the integer profits
constexpr int kBins = 2048;     // histogram bins, 32 per factor of two
constexpr int kCopies = 8;      // counters per bin
constexpr int kPlane = kBins + 32 / kCopies;
constexpr int kCoreMax = kRThreads;
constexpr int kMaxSearch = 40;  // evaluations of one price search
constexpr uint32_t kNone = 0xFFFFu;
constexpr int kChunks = kReduceActive / kRThreads;

// The active nodes a solve of k' chunks asks for above price 0.  Too few and
// the rung's price lies so near the final one that the gap passes it and the
// solve starts again lower; too many and every pass is longer.  Plans with
// k'/64 + 40, k'/16 + 160, k'/8 + 160: n = 50,000, k = 4,096 16.2, 16.4, 16.6 ms;
// k = 128 real-valued 13.4, 12.4, 12.3; conversations, 32 starts 64.0, 53.3, 54.2.
__host__ __device__ constexpr int64_t nodes_needed(int64_t kp) { return kp + kp / 16 + 160; }

// Bins of the entry widths: exact below 4, then four per factor of two.
constexpr int kWidthBins = 256;
__device__ __forceinline__ int width_bin(int64_t a) {
  if (a < 4) return (int)a;
  const int e = 63 - __builtin_clzll((unsigned long long)a);
  return 4 * (e - 1) + (int)((a >> (e - 2)) & 3);
}
__device__ __forceinline__ int64_t width_edge(int b) {  // least value in bin b
  return b < 4 ? b : (int64_t)(4 + (b & 3)) << (b / 4 - 1);
}

struct Red {  // block-wide scratch words in LDS
  double dsum[kRWaves];
  int64_t isum[kRWaves];
  uint32_t wsum[kRWaves];
  uint32_t vh[kWidthBins];
  int32_t bt;
  uint32_t core, forced;
  uint32_t used[kCoreMax / 32];  // core depths of the rows that are skipped to
  int64_t value;
  double price[kLadderRungs];
  int32_t count[kLadderRungs];
  int32_t lev[2 * kChunks];  // first and last level of each 1024 active nodes
};

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Barrier where only LDS is exchanged: global loads stay in flight across it.
// The fence waits for accesses that the compiler knows to be LDS (ds_*).  A
// pointer into LDS that has been through an integer is a generic one, its
// accesses are flat_* and the fence alone lets them pass the barrier; so LDS
// is addressed by offsets from its base, and the wait (lgkmcnt(0), vmcnt as
// it is) is also stated.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Exclusive prefix over the block of one count per thread; *total: the sum.
__device__ uint32_t block_scan(uint32_t c, uint32_t* wsum, uint32_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t x = c;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wv] = x;
  lds_barrier();
  uint32_t base = 0, t = 0;
#pragma unroll
  for (int k = 0; k < kRWaves; ++k) {
    const uint32_t v = wsum[k];
    base += k < wv ? v : 0u;
    t += v;
  }
  lds_barrier();
  *total = t;
  return base + x - c;
}

__device__ int64_t block_total(int64_t v, int64_t* part) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  lds_barrier();
  int64_t t = 0;
#pragma unroll
  for (int k = 0; k < kRWaves; ++k) t += part[k];
  lds_barrier();
  return t;
}

// ----------------------------------------------------------- ladder ----

// Prices of the rungs: the profits of rank c k', for these c (times 1/16).
// |S| at a price is between about 0.4 and 1 times the number of profits
// above it on prefix trees (profits that the other workers' copies leave
// under poor ancestors do not count), so the steps are small there.
// Launches of more than 16 chains take half as many steps, so that the blocks
// fit the chip at once.  The last ones are for gaps that are a large part of a
// price (small k').
__device__ constexpr int kRankLong[kLadderRungs] = {4,  11, 13, 15, 17, 19,  22, 25,
                                                    29, 34, 41, 50, 64, 100, 400};
__device__ constexpr int kRankShort[kLadderShort] = {9, 14, 18, 24, 34, 56, 150};

__device__ __forceinline__ int rung_rank16(int rung, int rungs) {
  return rungs == kLadderRungs ? kRankLong[rung] : kRankShort[rung];
}

// S_t for a ladder of prices t, one block per (chain, rung).  Profits come as
// the upper 32 bits of doubles, rounded up (profit keys).  Child sums are
// 32-bit fixed-point upper bounds in units of t / 2^u, so the result holds
// S_t: values are clipped at a height that leaves every ancestor positive
// (the clip exceeds one price per level).  Integer sums: the same bits
// whatever the order of the atomics.
// Bound by one block's passes over all nodes (histogram, up, down), in about
// equal parts issue and waits, and the barriers between levels: 48 us at
// n = 50,000, m = 16, 17 us at n = 10,000, 79 us on deep conversation trees of
// 50,000 (7 rungs, 32 chains).  The leaf passes take one value at a time: the
// ballots in them keep the compiler from unrolling.  Blocks of different rungs
// run side by side, so more rungs cost nothing until chains x rungs pass the
// 256 compute units.
// With `prep` set, one more block per chain sums the incumbent's value
// sum over T_h of p_h of a refinement update (what k_gains leaves in inc;
// real-valued costs: also the scale wsum, from the start's gwo).
template <bool F64>
__global__ void __launch_bounds__(kRThreads) k_ladder(ChainSet set, DevState d, int rungs,
                                                      int prep) {
  extern __shared__ int64_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  if (prep && (int)blockIdx.x >= set.count * rungs) {
    const int ci = blockIdx.x - set.count * rungs;
    ChainState* st = d.cs + set.slot[ci];
    const int64_t ps = set.src[ci], n = d.n;
    const uint8_t* th = d.tgt + (ps * d.m + set.worker[ci]) * n;
    const int64_t* p = d.profit + (int64_t)set.row[ci] * n;
    Red* red = (Red*)lds;
    int64_t acc = 0;
    double accf = 0.0;
#pragma unroll 8
    for (int64_t i = tid; i < n; i += kRThreads)
      if (th[i]) {
        if (F64) accf += __builtin_bit_cast(double, p[i]);
        else acc += p[i];
      }
    if (F64) {
      for (int o = 32; o > 0; o >>= 1) accf += __shfl_down(accf, o, 64);
      if (lane == 0) red->dsum[tid >> 6] = accf;
      __syncthreads();
      if (tid == 0) {
        double v = 0.0;
        for (int k = 0; k < kRWaves; ++k) v += red->dsum[k];
        st->inc = __builtin_bit_cast(int64_t, v);
        st->wsum = d.cs[ps].gwo;
      }
    } else {
      acc = block_total(acc, red->isum);
      if (tid == 0) st->inc = acc;
    }
    return;
  }
  const int wv = uniform(tid >> 6);
  const int ci = blockIdx.x / rungs, rung = blockIdx.x % rungs;
  const int64_t slot = set.slot[ci];
  if (!prep && d.cs[slot].skip) return;
  const int kp = set.kprime[ci];
  const int levels = d.levels, nlv = d.nlv, leaf0 = d.leaf0;
  const int nlw = nlv / 32, n64 = nlv / 64;
  Red* red = (Red*)lds;
  int32_t* lst = (int32_t*)((char*)lds + kReduceRedBytes);  // level starts, then leaf0
  uint32_t* bits = (uint32_t*)(lst + ((levels + 2) & ~1));  // (8-byte aligned)
  uint32_t* cs = bits + nlw;
  // The histogram comes first, kCopies counters per bin (in planes a few
  // banks apart): most profits fall into a few bins, and atomics of one wave
  // on one counter take turns.
  uint32_t* suf = cs;
  uint32_t* const sufc = suf + (lane % kCopies) * kPlane;
  const uint32_t* __restrict__ key = d.key_lv + (int64_t)set.row[ci] * nlv;
  const uint16_t* __restrict__ par = d.lvpar;
  for (int q = tid; q <= levels; q += kRThreads) lst[q] = d.lvtab[q];
  for (int b = tid; b < kPlane * kCopies; b += kRThreads) suf[b] = 0;
  int base = 1023 << 5;  // integer profits: from 1 up
  __syncthreads();
  // (padding slots have key 0: no profit)
  if (F64) {  // the 64 octaves below the largest profit
    uint32_t mx = 0;
#pragma unroll 8
    for (int i = tid; i < nlv; i += kRThreads) mx = max(mx, key[i]);
    for (int o = 32; o > 0; o >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, o, 64));
    if (lane == 0) red->wsum[wv] = mx;
    __syncthreads();
    for (int k = 0; k < kRWaves; ++k) mx = max(mx, red->wsum[k]);
    base = (int)(mx >> 15) - (kBins - 1);
    __syncthreads();
  }
  // Ranks of many hundreds are estimated from every fourth profit: the rungs
  // need not be exact (all profits: 17.15 against 16.4 ms a plan at n =
  // 50,000, m = 16, k = 4,096, 55.3 against 53.3 on conversations with 32
  // starts; below k' = 1,024 a sample would move the small ranks).
  const int every = kp >= 1024 ? 4 : 1;
#pragma unroll 8
  for (int i = tid * every + (tid & (every - 1)); i < nlv; i += kRThreads * every) {
    const uint32_t x = key[i];
    if (x) atomicAdd(sufc + max((int)(x >> 15) - base, 0), 1u);
  }
  lds_barrier();
  // the rung's price: the largest edge with at least `want` profits above
  const int64_t want = max((int64_t)1, (int64_t)rung_rank16(rung, rungs) * kp / (16 * every));
  {
    constexpr int per = kBins / kRThreads;
    uint32_t c = 0, h[per];
#pragma unroll
    for (int b = 0; b < per; ++b) {
      h[b] = 0;
#pragma unroll
      for (int k = 0; k < kCopies; ++k) h[b] += suf[k * kPlane + tid * per + b];
      c += h[b];
    }
    if (tid == 0) red->bt = 0;
    uint32_t tot;
    uint32_t run = block_scan(c, red->wsum, &tot);
    run = tot - run;  // profits in this thread's bins and above
#pragma unroll
    for (int b = 0; b < per; ++b) {
      const uint32_t above = run - h[b];
      if ((int64_t)run >= want && (int64_t)above < want) red->bt = tid * per + b;
      run = above;
    }
    __syncthreads();
  }
  const int bt = red->bt;
  const double t = bt <= 0 ? 0.0
                           : __builtin_bit_cast(double, (uint64_t)((uint32_t)(bt + base) << 15) << 32);
  const int clip = d.lv_clip;
  const int unit = t > 0.0 ? 1 << d.lv_bits : 0;
  const double inv = t > 0.0 ? (double)unit / t : 0.0;
  const double clipd = (double)(clip - 2);
  // p - t in units, rounded up (price 0: only whether there is a profit).
  // inv is infinite for prices below about 2^lv_bits / DBL_MAX: then every
  // profit is clipped, and no profit (padding slots among them), whose product
  // with inv would be NaN, stays worth nothing.
  auto up = [&](uint32_t x) -> int {
    if (t == 0.0) return x ? clip : 0;
    if (x == 0) return 2 - unit;
    return (int)fmin(__builtin_bit_cast(double, (uint64_t)x << 32) * inv, clipd) + 2 - unit;
  };
  for (int q = tid; q < leaf0; q += kRThreads) cs[q] = 0;
  __syncthreads();
  uint64_t* const bits64 = (uint64_t*)bits;
  auto put = [&](int i, uint64_t m) {  // the wave's 64 bits at slot i - lane
    if (lane == 0) bits64[i >> 6] = m;
  };
  // up: the leaves at once, then the levels from the deepest
  for (int i = leaf0 + tid; i < nlv; i += kRThreads) {
    const int v = up(key[i]);
    const uint32_t pr = par[i];
    put(i, __ballot(v > 0));
    if (v > 0 && pr != kNone) atomicAdd(cs + pr, (uint32_t)min(v, clip));
  }
  // (a thread's first node of the two levels above is loaded ahead)
  {
    uint32_t k0 = 0, p0 = kNone, k1 = 0, p1 = kNone;
    auto load = [&](int q, uint32_t& k, uint32_t& p) {
      const int i = q >= 0 ? min(lst[q] + tid, nlv - 1) : 0;
      k = key[i];
      p = par[i];
    };
    load(levels - 1, k0, p0);
    load(levels - 2, k1, p1);
    for (int q = levels - 1; q >= 0; --q) {
      const int end = lst[q + 1];
      uint32_t x = k0, pr = p0;
      k0 = k1;
      p0 = p1;
      load(q - 2, k1, p1);
      lds_barrier();
      for (int i = lst[q] + tid; i < end; i += kRThreads) {
        // (past the level's end: some later slot, unused)
        const uint32_t xn = key[min(i + kRThreads, nlv - 1)];
        const uint32_t pn = par[min(i + kRThreads, nlv - 1)];
        const int v = up(x) + (int)cs[i];
        put(i, __ballot(v > 0));
        if (v > 0 && pr != kNone) atomicAdd(cs + pr, (uint32_t)min(v, clip));
        x = xn;
        pr = pn;
      }
    }
  }
  // down: what hangs on positive ancestors
  {
    auto keep = [&](int i, uint32_t pr) {
      const uint64_t own = bits64[i >> 6];
      const uint32_t pw = bits[pr >> 5];  // (roots: some word in LDS)
      const uint64_t m = __ballot(pr == kNone || ((pw >> (pr & 31)) & 1u));
      put(i, own & m);
    };
    auto load = [&](int q) { return (uint32_t)par[q < levels ? min(lst[q] + tid, nlv - 1) : 0]; };
    uint32_t p0 = load(1), p1 = load(2);
    for (int q = 1; q < levels; ++q) {
      const int end = lst[q + 1];
      uint32_t pr = p0;
      p0 = p1;
      p1 = load(q + 2);
      lds_barrier();
      for (int i = lst[q] + tid; i < end; i += kRThreads) {
        const uint32_t pn = par[min(i + kRThreads, nlv - 1)];
        keep(i, pr);
        pr = pn;
      }
    }
    lds_barrier();
    for (int i = leaf0 + tid; i < nlv; i += kRThreads) keep(i, par[i]);
    lds_barrier();
  }
  uint32_t* out = d.lad_bits + ((int64_t)ci * kLadderRungs + rung) * nlw;
  for (int w = tid; w < nlw; w += kRThreads) out[w] = bits[w];
  uint32_t tot;
  const uint32_t run = block_scan(tid < n64 ? __popcll(bits64[tid]) : 0, red->wsum, &tot);
  if (tid < n64) d.lad_pre[((int64_t)ci * kLadderRungs + rung) * n64 + tid] = run;
  if (tid == 0) {
    d.lad_price[ci * kLadderRungs + rung] = t;
    d.lad_count[ci * kLadderRungs + rung] = (int32_t)tot;
  }
}

// ------------------------------------------------------------ solve ----

// Row words of the core DP: bit 0 forced (real-valued costs), bit 1 leaf
// (the skip operand is the previous row), bits 2..15 the slot the row is
// stored to (0: none), bits 16..31 the slot of the skip operand (0: the row
// past the end, all zero).
constexpr uint32_t kRowForced = 1u, kRowLeaf = 2u;

__device__ __forceinline__ double as_d(int64_t v) { return __builtin_bit_cast(double, v); }
__device__ __forceinline__ int64_t as_l(double v) { return __builtin_bit_cast(int64_t, v); }

__device__ __forceinline__ int64_t shr1(int64_t v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), 0x138, 0xf, 0xf, true);
  return (int64_t)((uint64_t)(uint32_t)hi << 32 | (uint32_t)lo);
}

__device__ __forceinline__ int64_t lane_of(int64_t v, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l);
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// The core DP of one wave, columns 0..64C-1 (lane l: columns lC .. lC+C-1),
// rows last to first; *out: the last row's value at column col.  Choice masks
// of core row r (its rank among the core rows): ch[r C + c].
// One dependent chain of rows: the words and profits of 64 rows are in
// registers (lane l: row base - l, the next 64 on their way), and only rows
// that skip past a subtree wait for LDS, their operand read one row ahead (the
// row just computed is never the next row's far operand: that one is a leaf).
// Forced rows that nothing skips to are one addition.  Reading each row's word
// and operand from LDS took about 120 ns a row, most of the solve at large k'
// where costs are real-valued: n = 50,000, m = 16, k = 4,096: k_reduce 633 ->
// 230 us per launch, at k = 128 124 -> 111; integer cores, which have no forced
// rows, stay where they were (84 and 87 us, 217 and 219).
template <int C, bool F64>
__device__ void core_dp(int rows, int core, const int64_t* rp, const uint32_t* rinfo,
                        int64_t* slots, uint64_t* ch, int col, int64_t* out) {
  const int lane = threadIdx.x & 63;
  int64_t D[C], skn[C];
#pragma unroll
  for (int c = 0; c < C; ++c) D[c] = skn[c] = slots[c * 64 + lane] = 0;
  auto far = [&](uint32_t in) {  // the row's skip operand
#pragma unroll
    for (int c = 0; c < C; ++c) skn[c] = slots[((in >> 16) * C + c) * 64 + lane];
  };
  uint32_t ri = 0;
  int64_t pi = 0;
  if (rows > 0) {
    ri = rinfo[max(rows - 1 - lane, 0)];
    pi = rp[max(rows - 1 - lane, 0)];
  }
  int cr = core;
  for (int base = rows - 1; base >= 0; base -= 64) {
    const int cnt = min(64, base + 1);
    const uint32_t w = ri;
    const int64_t q = pi;
    if (base >= 64) {
      ri = rinfo[max(base - 64 - lane, 0)];
      pi = rp[max(base - 64 - lane, 0)];
    }
    // forced, not stored
    const uint64_t plain =
        F64 ? __ballot(lane < cnt && (w & kRowForced) && (w & 0xFFFCu) == 0) : 0ull;
    bool ahead = false;  // row l's operand is in skn
    for (int l = 0; l < cnt;) {
      if (F64 && ((plain >> l) & 1u)) {
        const uint64_t rest = ~(plain >> l);
        const int end = l + (rest ? __builtin_ctzll(rest) : 64);
        for (; l < end; ++l) {
          const double p = as_d(lane_of(q, l));
#pragma unroll
          for (int c = 0; c < C; ++c) D[c] = as_l(p + as_d(D[c]));
        }
        ahead = false;
        continue;
      }
      const uint32_t in = (uint32_t)__builtin_amdgcn_readlane((int)w, l);
      const int64_t p = lane_of(q, l);
      if (F64 && (in & kRowForced)) {
        ahead = false;
#pragma unroll
        for (int c = 0; c < C; ++c) D[c] = as_l(as_d(p) + as_d(D[c]));
      } else {
        int64_t sk[C];
        if (in & kRowLeaf) {
#pragma unroll
          for (int c = 0; c < C; ++c) sk[c] = D[c];
        } else {
          if (!ahead) far(in);
#pragma unroll
          for (int c = 0; c < C; ++c) sk[c] = skn[c];
        }
        const uint32_t nx = l + 1 < cnt ? (uint32_t)__builtin_amdgcn_readlane((int)w, l + 1)
                                        : kRowLeaf;
        ahead = (nx & (kRowLeaf | kRowForced)) == 0;
        if (ahead) far(nx);
        --cr;
        const int64_t left = shr1(D[C - 1]);
        int64_t t[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const int64_t v = c == 0 ? left : D[c - 1];
          t[c] = F64 ? as_l(as_d(p) + as_d(v)) : p + v;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
          // non-negative doubles compare like their bit patterns
          const bool take = t[c] > sk[c] && (c > 0 || lane > 0);
          const uint64_t m = __ballot(take);
          if (lane == 0) ch[cr * C + c] = m;
          D[c] = take ? t[c] : sk[c];
        }
      }
      const uint32_t st = (in >> 2) & 0x3FFFu;
      if (st != 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) slots[(st * C + c) * 64 + lane] = D[c];
      }
      ++l;
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (lane == col / C && c == col % C) *out = D[c];
}

// The walk from (core row 0, column col): 64 core rows' masks and links are in
// registers; the positions of the rows taken are marked in sel.
template <int C>
__device__ void core_walk(int core, const uint64_t* ch, const uint16_t* cnx,
                          const uint32_t* cpos, int col, uint32_t* sel) {
  const int lane = threadIdx.x & 63;
  int r = 0, j = col;
  for (int b = 0; b < core && j > 0; b += 64) {
    if (r >= b + 64) continue;
    const int mine = min(b + lane, core - 1);
    uint64_t m[C];
#pragma unroll
    for (int c = 0; c < C; ++c) m[c] = ch[mine * C + c];
    const int nx = cnx[mine];
    uint64_t taken = 0;
    while (r < min(b + 64, core) && j > 0) {
      const int l = r - b;
      uint64_t w = m[0];
      if (C > 1) {
#pragma unroll
        for (int c = 1; c < C; ++c) w = (j & (C - 1)) == c ? m[c] : w;
      }
      const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)w, l);
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(w >> 32), l);
      const uint64_t row = (uint64_t)hi << 32 | lo;
      if ((row >> (j / C)) & 1u) {
        taken |= 1ull << l;
        ++r;
        --j;
      } else {
        r = __builtin_amdgcn_readlane(nx, l);
      }
    }
    if ((taken >> lane) & 1u) {
      const uint32_t q = cpos[b + lane];
      atomicOr(sel + (q >> 5), 1u << (q & 31));
    }
  }
}

// A solved update: its value, and the decision and marks k_backtrack makes
// after a sweep (real-valued costs: the early rejection; the decision itself
// is k_gexact_final's).
template <bool F64>
__device__ void finish_update(ChainState* st, const DevState& d, int h, int kp, int mode,
                              int64_t dpval) {
  st->dpval = dpval;
  st->solved = 1;
  st->dirty[h >> 5] &= ~(1u << (h & 31));
  if (F64) {
    st->rejected = mode == kModeRefine &&
                           early_reject_f64(as_d(dpval), as_d(st->inc), as_d(st->wsum), d.m, kp,
                                            d.n, d.eps)
                       ? 1
                       : 0;
    st->wsum = 0;
  } else if (mode == kModeGreedy || dpval > st->inc) {
    st->accept = 1;
    if (mode == kModeRefine) st->accepts += 1;
    for (int q = 0; q < 8; ++q) st->dirty[q] |= q == (h >> 5) ? ~(1u << (h & 31)) : ~0u;
  }
  st->inc = 0;
}

// One block per chain: list, price search, entry widths, core, DP and walk.
// Bound by the chain of these phases, each 10 to 20 us of one block's waits
// (barriers, LDS, the one wave of the core DP), with 8 to 32 of 256 compute
// units in use; 8 (real-valued) to 28 vector registers spill (36 to 116 bytes
// of scratch a lane at 16 waves a block).  78 us a launch at
// n = 50,000, k = 4,096 (the sweep and walk it replaces: 2,160 + 320 us), 51 us
// at n = 10,000, k = 1,024 (430 us), 83 us real-valued at k = 128 (1,890 us).
template <bool F64>
__global__ void __launch_bounds__(kRThreads) k_reduce(ChainSet set, DevState d, int mode,
                                                      int lds_bytes, int rungs) {
  extern __shared__ int64_t lds[];
  const int tid = threadIdx.x;
  const int ci = blockIdx.x;
  const int64_t slot = set.slot[ci];
  ChainState* st = d.cs + slot;
  if (st->skip) {
    if (tid == 0) {
      st->accept = 0;
      st->inc = 0;
    }
    return;
  }
  const int h = set.worker[ci];
  // (read ahead of the first barrier: finish_update clears them)
  const int64_t inc = st->inc, wsum = st->wsum;
  const int n = d.n, nw = (n + 31) / 32, n64 = d.nlv / 64;
  const int kp = set.kprime[ci];
  const int64_t* __restrict__ prof = d.profit + (int64_t)set.row[ci] * n;
  // the active nodes, leaves first, then the deepest level: position, parent's
  // index | level << 16 (leaves: d.levels), integer profit (an entry is
  // written and read by one thread)
  uint32_t* apos = d.lad_list + ci * (int64_t)(4 * kReduceActive);
  uint32_t* amd = apos + kReduceActive;
  int64_t* aq = (int64_t*)(amd + kReduceActive);

  Red* red = (Red*)lds;
  uint32_t* sel = (uint32_t*)((char*)lds + kReduceRedBytes);  // selection, n bits
  const int woff = (kReduceRedBytes + 4 * nw + 15) & ~15;
  int64_t* W = (int64_t*)((char*)lds + woff);
  const int wbytes = lds_bytes - woff;
  const int acap = min(kReduceActive, wbytes / 8 - 4);

  if (tid == 0) {  // undecided, until solved here or swept
    st->solved = 0;
    st->accept = 0;
    st->rejected = 1;
  }
  if (kp <= 0) return;
  double* price = red->price;
  int32_t* count = red->count;
  if (tid < rungs) {
    price[tid] = d.lad_price[ci * kLadderRungs + tid];
    count[tid] = d.lad_count[ci * kLadderRungs + tid];
  }
  __syncthreads();
  // the highest rung with clearly more than k' nodes, else price 0
  const int need = (int)nodes_needed(kp);
  int j = 0;
  while (j < rungs - 1 && count[j] < need && price[j] > 0.0) ++j;
  const int nwords = d.npad / 32;
  uint32_t* selw = d.sel + slot * nwords;

  for (;;) {  // again from a lower rung if the gap turns out to need it
    const double t = price[j];
    const int A = count[j];
    if (A > acap || (A < need && t > 0.0)) return;
    if (A == 0) {  // price 0, no profit: nothing is strictly better than skipping
      for (int w = tid; w < nwords; w += kRThreads) selw[w] = 0;
      if (tid == 0) finish_update<F64>(st, d, h, kp, mode, 0);
      return;
    }
    const int chunks = (A + kRThreads - 1) / kRThreads;

    // --------------------------------------------------- active nodes --
    {
      uint32_t* list = (uint32_t*)W;
      uint64_t* lb = (uint64_t*)(list + kReduceActive);
      uint32_t* lp = (uint32_t*)(lb + n64);
      if (tid < n64) {
        const int64_t o = ((int64_t)ci * kLadderRungs + j) * n64 + tid;
        const uint64_t m = ((const uint64_t*)d.lad_bits)[o];
        int x = A - 1 - (int)d.lad_pre[o];
        lb[tid] = m;
        lp[tid] = (uint32_t)x;  // active index of the group's first node
        // (a thread per 64 slots: a wave-wide compaction per group took twice
        // as long, 800 groups each paying its LDS latency)
        for (uint64_t r = m; r; r &= r - 1) list[x--] = (uint32_t)(64 * tid + __builtin_ctzll(r));
      }
      lds_barrier();
      double total = 0.0;
#pragma unroll 2
      for (int x = tid; x < A; x += kRThreads) {
        const uint32_t s = list[x];
        const uint32_t pd = d.lvpos[s], pr = d.lvpar[s];
        const int64_t p = prof[pd & 0xFFFFFFu];
        uint32_t ps = kNone;
        if (pr != kNone)
          ps = lp[pr >> 6] - __popcll(lb[pr >> 6] & ((1ull << (pr & 63)) - 1u));
        const int lv = min((int)(pd >> 24), d.levels);  // leaves: below every level
        apos[x] = pd & 0xFFFFFFu;
        amd[x] = ps | (uint32_t)lv << 16;
        aq[x] = p;
        total += F64 ? as_d(p) : (double)p;
        if ((x & (kRThreads - 1)) == 0) red->lev[2 * (x / kRThreads)] = lv;
        if (x == A - 1 || (x & (kRThreads - 1)) == kRThreads - 1)
          red->lev[2 * (x / kRThreads) + 1] = lv;
      }
      for (int o = 32; o > 0; o >>= 1) total += __shfl_down(total, o, 64);
      if ((tid & 63) == 0) red->dsum[tid >> 6] = total;
      __syncthreads();
    }
    double total = 0.0;
    for (int k = 0; k < kRWaves; ++k) total += red->dsum[k];
    if (!(total < 1.7976931348623157e308) || (!F64 && total >= 9.2e18)) return;
    // integer profits: p >> shift; real-valued: trunc(p 2^scale)
    const int lg = ilogb(total * (1.0 + 0x1p-20));
    const int shift = max(0, lg + 1 - kValueBits);
    const int scale = F64 ? kValueBits - 1 - lg : -shift;
    const int64_t qerr = (F64 || shift > 0) ? kp : 0;  // units UB can be low by
    auto quant = [&](int64_t p) -> int64_t {
      return F64 ? (int64_t)ldexp(as_d(p), scale) : p >> shift;
    };
    // a price in these units, rounded up
    auto price_q = [&](double v) -> int64_t {
      return (int64_t)fmin(ceil(ldexp(v, scale)), 0x1p48);
    };
    const int64_t tq = price_q(t);
    if (F64 || shift > 0)
      for (int x = tid; x < A; x += kRThreads) aq[x] = quant(aq[x]);

    // --------------------------------------------------- price search --
    // f(l) = |S(l)| falls with l; find a small l with f(l) <= k'.  The rungs'
    // counts bracket it (to be confirmed); regula falsi (Illinois), which is
    // quick where f falls in small steps.  UB(l) = l k' + rootsum is convex
    // and piecewise linear with slope k' - f(l), so where both ends are known
    // every other price is where their tangents meet: exact where one subtree
    // of many nodes joins at once, which a search on f alone would bisect.
    // The tangents also show when UB can fall by at most 2^-9 of the price
    // below the end hi: then hi will do.
    int64_t* cw = W;  // child sums by active index, then two root words
    int64_t lam = 0, rootsum = 0;
    {
      int jl = 0;  // the highest rung with more than k' nodes
      while (jl < j && count[jl] <= kp) ++jl;
      int64_t lo = price_q(price[jl]), hi;
      double ylo = max(count[jl] - kp, 1), yhi = -(double)kp;
      bool vhi = false;
      int fhi = 0, flo = 0;
      if (jl > 0) {
        hi = max(price_q(price[jl - 1]), lo + 2);
        yhi = min(count[jl - 1] - kp, -1);
      } else {
        hi = price[0] > 0.0 ? 2 * lo + 2 : price_q(total) + 2;
      }
      bool zero = t == 0.0 && jl == j;  // price 0 itself may be the one
      bool last = false;
      bool vlo = false;
      int side = 0;
      int64_t Llo = 0, Lhi = 0;
      uint32_t parity = 0;
      for (int it = 0;; ++it) {
        int64_t l;
        if (last) {
          l = hi;
        } else if (zero) {
          l = 0;
        } else if (hi - lo <= 1) {
          l = hi;
        } else if (vlo && vhi && (it & 1)) {
          const int64_t w = hi - lo;
          const double x = ceil((double)(Lhi - Llo - (int64_t)(kp - fhi) * w) /
                                (double)(fhi - flo));
          l = lo + min(max((int64_t)x, (int64_t)1), w - 1);
        } else {
          l = lo + (int64_t)((double)(hi - lo) * (ylo / (ylo - yhi)));
          l = min(max(l, lo + 1), hi - 1);
        }
        if (it >= kMaxSearch && !last) {
          if (!vhi) return;
          last = true;
          l = hi;
        }
        // |S| and the sum over roots of max(V, 0) at price l
        parity ^= 1u;
        for (int x = tid; x < A; x += kRThreads) cw[x] = 0;
        if (tid == 0) cw[acap + parity] = 0;
        int64_t qa = tid < A ? aq[tid] : 0, qb = 0;
        uint32_t ma = tid < A ? amd[tid] : 0xFFFF0000u, mb = 0xFFFF0000u;
        lds_barrier();
        int cur = uniform(red->lev[0]);
        for (int u = 0; u < chunks; ++u) {
          const int x = tid + kRThreads * u;
          const int64_t q = qa;
          const uint32_t md = ma;
          mb = 0xFFFF0000u;
          if (x + kRThreads < A) {
            qb = aq[x + kRThreads];
            mb = amd[x + kRThreads];
          }
          const int l0 = uniform(red->lev[2 * u]), l1 = uniform(red->lev[2 * u + 1]);
          for (int dd = l0; dd >= l1; --dd) {
            if (dd != cur) {  // the levels below are complete
              lds_barrier();
              cur = dd;
            }
            if ((int)(md >> 16) == dd) {
              const int64_t w = (q - l) * (1 << kSizeBits) + 1 + cw[x];
              const uint32_t ps = md & 0xFFFFu;
              if ((w >> kSizeBits) > 0)
                atomicAdd((unsigned long long*)&cw[ps == kNone ? acap + parity : ps],
                          (unsigned long long)w);
            }
          }
          qa = qb;
          ma = mb;
        }
        lds_barrier();
        const int64_t root = cw[acap + parity];
        const int fsize = (int)((uint32_t)root & ((1u << kSizeBits) - 1));
        rootsum = root >> kSizeBits;
        lam = l;
        if (last) break;
        const int miss = fsize - kp;
        if (miss <= 0) {
          hi = l;
          fhi = fsize;
          Lhi = l * kp + rootsum;
          vhi = true;
          if (zero || miss == 0) break;
          yhi = miss;
          if (side < 0) ylo *= 0.5;
          side = -1;
        } else {
          if (l == hi) {  // the rung above was no upper bound
            hi = l + max(l / 4, (int64_t)1);
            yhi = -(double)kp;
            vhi = false;
          }
          lo = l;
          flo = fsize;
          Llo = l * kp + rootsum;
          vlo = true;
          ylo = miss;
          if (side > 0) yhi *= 0.5;
          side = 1;
        }
        zero = false;
        if (vhi) {
          // how far below hi the tangents meet (the bracket, if only hi is
          // known)
          int64_t w = hi - lo;
          if (vlo && w > 1)
            w -= min((int64_t)ceil((double)(Lhi - Llo - (int64_t)(kp - fhi) * w) /
                                   (double)(fhi - flo)),
                     w);
          if (hi - lo <= 1 || (double)(kp - fhi) * (double)w * 512.0 <= (double)hi) {
            if (lam == hi) break;
            last = true;
          }
        }
      }
    }
    const int64_t ub = lam * kp + rootsum + qerr;
    if (mode == kModeRefine) {
      // no set can be worth more than the incumbent: rejected as it stands
      // (real-valued: only if the early test holds with the upper bound in
      // place of the value)
      bool reject;
      int64_t bound;
      if (!F64) {
        bound = ub <= (INT64_MAX >> shift) ? ub << shift : INT64_MAX;
        reject = bound <= inc;
      } else {
        const double v = ldexp((double)ub, -scale) * (1.0 + (kp + 8.0) * 0x1p-52);
        bound = as_l(v);
        reject = early_reject_f64(v, as_d(inc), as_d(wsum), d.m, kp, n, d.eps);
      }
      if (reject) {
        if (tid == 0) finish_update<F64>(st, d, h, kp, mode, bound);
        return;
      }
    }

    // ----------------------------------------------------------- core --
    // Entry width of each node, from the roots down, in place of its child
    // sum: > 0 in S, the least V on its ancestor path (in the core iff at
    // most the width, else forced); < 0 outside, -1 - the largest -V on the
    // path (in the core iff that is at most the width).
    if (tid < kWidthBins) red->vh[tid] = 0;
    {
      int cur = uniform(red->lev[2 * chunks - 1]);
      int64_t qa = 0;
      uint32_t ma = 0;
      const int xl = tid + kRThreads * (chunks - 1);
      if (xl < A) {
        qa = aq[xl];
        ma = amd[xl];
      }
      for (int u = chunks - 1; u >= 0; --u) {
        const int x = tid + kRThreads * u;
        const int64_t q = qa;
        const uint32_t md = x < A ? ma : 0xFFFF0000u;
        if (u > 0) {
          qa = aq[x - kRThreads];
          ma = amd[x - kRThreads];
        }
        const int l0 = uniform(red->lev[2 * u]), l1 = uniform(red->lev[2 * u + 1]);
        for (int dd = l1; dd <= l0; ++dd) {
          if (dd != cur) {
            lds_barrier();
            cur = dd;
          }
          if ((int)(md >> 16) == dd) {
            const int64_t V = ((q - lam) * (1 << kSizeBits) + 1 + cw[x]) >> kSizeBits;
            const uint32_t ps = md & 0xFFFFu;
            const int64_t ep = ps == kNone ? INT64_MAX : cw[ps];
            int64_t e;
            if (ep < 0) e = V > 0 ? ep : min(ep, V - 1);
            else e = V > 0 ? min(ep, V) : V - 1;
            cw[x] = e;
          }
        }
      }
      lds_barrier();
    }
    // nodes that are not active stay out while gap <= dmax
    const int64_t dmax = t == 0.0 ? INT64_MAX : max(lam - tq - 1, (int64_t)0);
    // numbers of nodes by entry width (four bins a factor of two), up to half a price (or a
    // few of the units the profits lose)
    const int64_t cutoff = max(lam >> 1, 4 * qerr + 1);
    for (int x = tid; x < A; x += kRThreads) {
      const int64_t e = cw[x], a = e < 0 ? -1 - e : e;
      if (a < cutoff) atomicAdd(&red->vh[width_bin(a)], 1u);
    }
    __syncthreads();
    // the largest width at a bin's end, below the cutoff, with at most `limit`
    // nodes
    auto widest = [&](uint32_t limit) -> int64_t {
      const int b = 4 * (tid & 63);
      uint32_t c[4], x = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) x += c[e] = red->vh[b + e];
      uint32_t y = x;
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t z = __shfl_up(y, o, 64);
        if ((tid & 63) >= o) y += z;
      }
      y -= x;
      int top = -1;  // a prefix of the bins fits
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y += c[e];
        if (y <= limit && b + e < kWidthBins - 8 && width_edge(b + e + 1) - 1 < cutoff)
          top = b + e;
      }
      const uint64_t m = __ballot(top >= 0);
      if (m == 0) return 0;
      const int w = __builtin_amdgcn_readlane(top, 63 - __builtin_clzll(m));
      return width_edge(w + 1) - 1;
    };
    int64_t width = min(dmax, widest(64));
    if (lam == 0) width = 0;
    // LDS after the child sums (the core is small: they stay for a second,
    // wider one)
    char* const X = (char*)(W + A);
    const int xbytes = wbytes - 8 * A;
    bool lower = false;
    for (int attempt = 0; attempt < 4 && !lower; ++attempt) {
      if (tid == 0) red->core = red->forced = 0;
      if (tid < kCoreMax / 32) red->used[tid] = 0;
      for (int w = tid; w < nw; w += kRThreads) sel[w] = 0;
      int off = 0;
      auto take = [&](int64_t bytes) {
        char* p = X + off;
        off = (int)min((int64_t)1 << 30, off + ((bytes + 15) & ~(int64_t)15));
        return p;
      };
      uint32_t* cun = (uint32_t*)take(4 * kCoreMax);  // core nodes as found
      if (off > xbytes) return;
      __syncthreads();
      // core nodes (any order); forced ones go to the selection, their value
      // into the base
      int64_t base = 0;
      uint32_t forced_mine = 0;
#pragma unroll 4
      for (int x = tid; x < A; x += kRThreads) {
        const int64_t e = cw[x], p = aq[x];
        const uint32_t q = apos[x];
        const bool core = e < 0 ? -1 - e <= width : e <= width;
        if (core) {
          const uint32_t c = atomicAdd(&red->core, 1u);
          if (c < (uint32_t)kCoreMax) cun[c] = q;
        } else if (e > 0) {
          atomicOr(sel + (q >> 5), 1u << (q & 31));
          ++forced_mine;
          if (!F64) base += shift == 0 ? p : prof[q];
        }
      }
      for (int o = 32; o > 0; o >>= 1) forced_mine += __shfl_down(forced_mine, o, 64);
      if ((tid & 63) == 0 && forced_mine) atomicAdd(&red->forced, forced_mine);
      base = block_total(base, red->isum);
      const int R = (int)red->core, forced = (int)red->forced;
      const int K = min(kp - forced, R);  // forced nodes are in S: at most k'
      if (R > kCoreMax || K < 0 || K > 255) return;
      const int C = K < 64 ? 1 : K < 128 ? 2 : 4;
      const int rows = F64 ? R + forced : R;
      uint32_t* cpos = (uint32_t*)take(4 * R);
      uint32_t* cend = (uint32_t*)take(4 * R);
      uint16_t* cnx = (uint16_t*)take(2 * R);
      uint16_t* cdep = (uint16_t*)take(2 * R);
      uint64_t* ch = (uint64_t*)take(8 * R * C);
      int64_t* rp = (int64_t*)take(8ll * rows);
      uint32_t* rinfo = (uint32_t*)take(4ll * rows);
      // real-valued: the rows' positions as a bitmap, and its prefix
      uint32_t* ib = F64 ? (uint32_t*)take(4 * nw) : sel;
      uint32_t* ip = F64 ? (uint32_t*)take(4 * nw) : sel;
      if (off > xbytes) return;
      // each core node: rank, next core row, and core depth (the core rows
      // before it whose subtree holds it)
      uint32_t q = 0, qe = 0, rk = 0, nx = 0, dep = 0;
      if (tid < R) {
        q = cun[tid];
        qe = (uint32_t)d.nextpos[q];
        cend[tid] = qe;
      }
      if (F64)
        for (int w = tid; w < nw; w += kRThreads) ib[w] = sel[w];
      for (int r = tid; r < rows; r += kRThreads) rinfo[r] = 0;
      __syncthreads();
      if (tid < R) {
#pragma unroll 4
        for (int a = 0; a < R; ++a) {
          const uint32_t qa = cun[a], ea = cend[a];
          rk += qa < q;
          nx += qa < qe;
          dep += qa < q && ea > q;
        }
        cpos[rk] = q;
        cnx[rk] = (uint16_t)nx;
        cdep[rk] = (uint16_t)dep;
        if (F64) atomicOr(ib + (q >> 5), 1u << (q & 31));
      }
      __syncthreads();
      if (F64) {
        const int per = (nw + kRThreads - 1) / kRThreads;
        const int w0 = tid * per, w1 = min(w0 + per, nw);
        uint32_t c = 0, tot;
        for (int w = w0; w < w1; ++w) c += __popc(ib[w]);
        uint32_t run = block_scan(c, red->wsum, &tot);
        for (int w = w0; w < w1; ++w) {
          ip[w] = run;
          run += __popc(ib[w]);
        }
        __syncthreads();
      }
      auto row_of = [&](uint32_t at) -> int {  // rows before position `at`
        return at >= (uint32_t)n
                   ? rows
                   : (int)(ip[at >> 5] + __popc(ib[at >> 5] & ((1u << (at & 31)) - 1u)));
      };
      // Row words.  A row is stored if some earlier core row that is no leaf
      // skips to it, in the slot of its core depth: between such a row and its
      // readers every other stored row lies below the reader, so it is deeper.
      // Forced rows have no core ancestor (depth 0).  Slots are numbered by
      // the depths that are in use.
      int it = 0, nit = 0;
      uint32_t td = kNone;  // depth of the row this one skips to
      if (tid < R) {
        it = F64 ? row_of(q) : (int)rk;
        nit = F64 ? row_of(qe) : (int)nx;
        rp[it] = prof[q];
        if (nit != it + 1 && nit < rows) {
          // the target (the first row at or past the subtree's end) is a core
          // row iff it is the first core row there
          td = (int)nx < R && (!F64 || row_of(cpos[nx]) == nit) ? cdep[nx] : 0u;
          atomicOr(&red->used[td >> 5], 1u << (td & 31));
        }
      }
      lds_barrier();
      int nslots = 1;  // the zero row
      uint32_t sd = 0;
      for (int w = 0; w < kCoreMax / 32; ++w) {
        const uint32_t m = red->used[w];
        if (w < (int)(td >> 5)) sd += __popc(m);
        nslots += __popc(m);
      }
      int64_t* slots = (int64_t*)take((int64_t)nslots * C * 512);
      if (off > xbytes) return;
      if (tid < R) {
        uint32_t info = nit == it + 1 ? kRowLeaf : 0u;
        if (td != kNone) {
          sd += __popc(red->used[td >> 5] & ((1u << (td & 31)) - 1u)) + 1u;
          info = sd << 16;
          atomicOr(&rinfo[nit], sd << 2);
        }
        atomicOr(&rinfo[it], info);
      }
      if (F64) {
        for (int x = tid; x < A; x += kRThreads)
          if (cw[x] > width) {
            const uint32_t at = apos[x];
            const int it = row_of(at);
            rp[it] = prof[at];
            atomicOr(&rinfo[it], kRowForced);
          }
      }
      __syncthreads();
      if (tid < 64) {
        if (C == 1) core_dp<1, F64>(rows, R, rp, rinfo, slots, ch, K, &red->value);
        else if (C == 2) core_dp<2, F64>(rows, R, rp, rinfo, slots, ch, K, &red->value);
        else core_dp<4, F64>(rows, R, rp, rinfo, slots, ch, K, &red->value);
      }
      __syncthreads();
      const int64_t value = F64 ? red->value : base + red->value;
      int64_t gap;
      if (F64) {
        // the value's integer units, low by what k' roundings can add
        const double v = as_d(value);
        if (!(v < 1.7976931348623157e308)) return;
        gap = ub - (int64_t)ldexp(v - v * ((kp + 8.0) * 0x1p-52), scale) + 1;
      } else {
        gap = ub - (value >> shift);
      }
      if (gap <= width) {
        if (tid < 64) {
          if (C == 1) core_walk<1>(R, ch, cnx, cpos, K, sel);
          else if (C == 2) core_walk<2>(R, ch, cnx, cpos, K, sel);
          else core_walk<4>(R, ch, cnx, cpos, K, sel);
        }
        __syncthreads();
        for (int w = tid; w < nwords; w += kRThreads) selw[w] = w < nw ? sel[w] : 0u;
        if (tid == 0) finish_update<F64>(st, d, h, kp, mode, value);
        return;
      }
      // wider: the gap itself, except that a first core's gap may only show
      // how poor its value is: then to at most 320 nodes
      const int64_t next = widest(320);
      const int64_t want = attempt == 0 && gap > next && next > width ? next : gap;
      if (width >= dmax) lower = true;
      else width = min(want, dmax);
    }
    if (!lower) return;
    int jn = j + 1;
    while (jn < rungs && price[jn] > 0.0 && count[jn] < A + A / 2) ++jn;
    if (jn >= rungs) return;
    j = jn;
    __syncthreads();
  }
}

}  // namespace

// Dynamic LDS the two kernels need at least on a tree of n nodes, nlv
// level-order slots, `levels` levels and leaf0 slots of internal nodes.
size_t ladder_lds(int32_t nlv, int32_t levels, int32_t leaf0) {
  return kReduceRedBytes + 4 * ((size_t)levels + 2) + (size_t)nlv / 8 +
         4 * (size_t)std::max<int32_t>(kPlane * kCopies, leaf0) + 16;
}

size_t reduce_lds_min(int32_t n, int32_t nlv, int32_t levels, int32_t leaf0) {
  const size_t nw = ((size_t)n + 31) / 32;
  const size_t solve = kReduceRedBytes + 4 * nw + 16 + 4 * (size_t)kReduceActive +
                       12 * (size_t)nlv / 64 + 64;
  return std::max(solve, ladder_lds(nlv, levels, leaf0));
}

int32_t reduce_reach(int32_t n, int f64, int lds) {
  const int64_t nw = ((int64_t)n + 31) / 32;
  const int64_t wbytes = lds - ((kReduceRedBytes + 4 * nw + 15) & ~(int64_t)15);
  const int64_t acap = std::min<int64_t>(kReduceActive, wbytes / 8 - 4);
  if (n <= acap) return n;
  auto fits = [&](int64_t kp) {
    const int64_t a = nodes_needed(kp);
    // child sums, core nodes as found, one row of the core's table;
    // real-valued costs: a row per forced node and the rows' bitmaps
    return a <= acap &&
           8 * a + 4 * kCoreMax + 512 + (f64 ? 12 * kp + 8 * nw : 0) <= wbytes;
  };
  int64_t lo = 0, hi = n;  // fits(lo)
  while (lo < hi) {
    const int64_t k = (lo + hi + 1) / 2;
    if (fits(k)) lo = k;
    else hi = k - 1;
  }
  return (int32_t)lo;
}

hipError_t launch_incumbents(const ChainSet& set, const DevState& d, hipStream_t st) {
  if (set.count == 0) return hipSuccess;
  if (d.f64)
    hipLaunchKernelGGL(k_ladder<true>, dim3(set.count), dim3(kRThreads), kReduceRedBytes, st, set,
                       d, 0, 1);
  else
    hipLaunchKernelGGL(k_ladder<false>, dim3(set.count), dim3(kRThreads), kReduceRedBytes, st, set,
                       d, 0, 1);
  return hipGetLastError();
}

hipError_t launch_reduce(const ChainSet& set, const DevState& d, int mode, int prep, int lds,
                         hipStream_t st) {
  static_assert(sizeof(Red) <= kReduceRedBytes, "scratch words");
  static_assert(kLadderSlots <= 64 * kRThreads, "one thread per 64 slots");
  if (set.count == 0) return hipSuccess;
  if (!d.key_lv || !d.lvpos || !d.lvpar || !d.lvtab || !d.lad_bits || !d.lad_pre ||
      !d.lad_price || !d.lad_count || !d.lad_list ||
      reduce_lds_min(d.n, d.nlv, d.levels, d.leaf0) > (size_t)lds)
    return hipErrorInvalidValue;
  const size_t lad = ladder_lds(d.nlv, d.levels, d.leaf0);
  const int rungs = set.count <= 16 ? kLadderRungs : kLadderShort;
  const dim3 grid((unsigned)(set.count * (rungs + (prep ? 1 : 0))));
  if (d.f64) {
    hipLaunchKernelGGL(k_ladder<true>, grid, dim3(kRThreads), lad, st, set, d, rungs, prep);
    hipLaunchKernelGGL(k_reduce<true>, dim3(set.count), dim3(kRThreads), lds, st, set, d, mode,
                       lds, rungs);
  } else {
    hipLaunchKernelGGL(k_ladder<false>, grid, dim3(kRThreads), lad, st, set, d, rungs, prep);
    hipLaunchKernelGGL(k_reduce<false>, dim3(set.count), dim3(kRThreads), lds, st, set, d, mode,
                       lds, rungs);
  }
  return hipGetLastError();
}

}  // namespace pp
