// Work plan of the sparse attention and the merge of its KV splits
// (Sec. 3.3 Eq. split and Eq. cost).
//
// plan_kernel runs once per call after the kept lists exist. The cost of a
// unit (sequence b, KV head h, query block I) is proportional to its number
// of 64-key steps (Eq. cost): two per kept block, one per 64 corrected
// blocks, plus a fixed per-item share. In the cost-balanced mode (splits ==
// 0) every unit whose cost exceeds a step budget S is cut into
// U = ceil(cost / S) parts (at most kMaxRowSplits); S is one resident
// workgroup's share of the call (never less than a minimum, and large enough
// for the partial-output capacity of the workspace). A fixed count n >= 1 cuts
// every unit into n.
// Part u of a unit walks kept-list positions [u ceil(T/U), min((u+1)
// ceil(T/U), T)) of its T kept blocks and the u-th of U equal ranges of the
// pruned blocks (Eq. split). The plan is an item table by decreasing cost
// class (units without queries left out), per-unit {U, first partial slot},
// and the list of units with U > 1.
//
// Heaviest first: the attention's workgroups take items in table order, so a
// heavy item near the end of the table runs on while the others idle. The
// selected blocks of the heads of one query block differ by up to 20x, so the
// order of decreasing query block left the chip idle for 40% of a chunked
// call: an 8K bf16 chunk after 56K tokens 1.42 -> 1.00 ms, four ragged fp8
// extends 0.94 -> 0.70 ms, a 32K prompt 1.667 -> 1.638 ms. kClasses linear
// cost classes come within 1% of a full sort; within a class the items keep
// the order of decreasing query block. Where no unit weighs much
// against a workgroup's share the order stays that of the query blocks, which
// mixes heavy and light items on the chip at any time (sorted: 128K fp8 5.20 ->
// 5.27 ms), and so does it for 4-wave workgroups, two of which share a compute
// unit and level each other (128-row tiles at 32K 1.03 -> 1.23 ms when
// sorted). A budget of one share needs the fewest parts that still level the
// load: a quarter of it costs more in partial outputs.
//
// Latency-bound: all of it lies between the selection and the attention. Every
// workgroup computes all costs (coalesced over the counts, kept in LDS) and
// the class histogram, and writes the table entries of its own range of
// units, so no workgroup waits for another. Past kCostCache units the costs are
// computed again where they are needed: for all units in every round of the
// budget and in the histogram, for its own range in the entries. The last is the
// longest part, so that as many workgroups as otherwise share it (131072 units
// 179 us, 234 with 4 of them; 36864 62 and 82).
//
// combine_kernel merges the parts of every split unit with the log-sum-exp
// weights: M = max_u m_u, w_u = 2^(m_u - M), O = c_v sum_u w_u o_u /
// sum_u w_u l_u, LSE = (M + log2 sum_u w_u l_u - offset) ln 2. Parts that saw
// no key have m_u = -inf and weight 0. It is HBM-bound (U x 520 bytes read
// and 256 written per packed row) and persistent over (split unit, 8-row
// group) pairs.
#include <atomic>
#include <algorithm>

#include "kernels.h"

namespace fp2 {

namespace {

constexpr float kLn2 = 0.69314718055994530942f;
constexpr int kPlanThreads = 1024;   // threads of a plan workgroup
constexpr int kPlanThreadsFew = 256;   // the same for at most kPlanFewUnits units: shorter barriers
constexpr int kPlanFewUnits = 1024;
// Smallest step budget of an item: below it the parts' fixed work, partial
// outputs and merge cost more than the cut saves. bf16 calls whose units would
// leave most compute units without an entry take 8 (18 tokens after 1000 51 -> 45
// us, 100 after 60000 98 -> 91, 18 after 500 42 -> 45). fp8 calls do not: their
// steps are shorter (40 tokens after 1500 43.0 us, cut to 8 steps 45.2; 600 with
// 4/1 heads 38.1 and 41.2; 18 after 1000 47.9 and 44.8), and every cut rounds
// their probabilities against one more reference.
constexpr int kMinSplitSteps = 16;
constexpr int kMinSplitStepsFewBf16 = 8;
constexpr int kItemSteps = 2;        // fixed per-item cost (query load, set-up), in steps
constexpr int kMaxRowSplits = 64;    // two parts per lane of the combine's half-wave
constexpr int kClasses = 32;         // cost classes of the item order
// Items of 8-wave workgroups (one per compute unit) are put in order of cost
// when the heaviest unit exceeds this part of a workgroup's share of the call.
// The order of query blocks shares more K/V in the caches, which weighs more
// in fp8 (10.7K tokens, heaviest 1.24 shares: sorted 254 -> 260 us; bf16 30K,
// 0.83 shares: 786 -> 767 us).
constexpr double kSortAboveBf16 = 0.6, kSortAboveFp8 = 1.5;
constexpr int kCostCache = 32768;    // units whose costs a plan workgroup keeps in LDS (64 KiB)
constexpr int kPlanUnits = 512;      // units whose entries a plan workgroup writes (at least)
constexpr int kPlanGroups = 32;      // plan workgroups (at most)
constexpr uint32_t kNoCost = 0xffffu;  // a unit without queries; real costs are below 2 * 8192 + 131

// Sum of v and maximum of m over the TH threads of the workgroup.
template <int TH>
__device__ void block_sum_max(double& v, int& m, double* shd, int* shi) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int o = 32; o > 0; o >>= 1) {
    v += __shfl_xor(v, o, 64);
    m = max(m, __shfl_xor(m, o, 64));
  }
  __syncthreads();
  if (lane == 0) {
    shd[w] = v;
    shi[w] = m;
  }
  __syncthreads();
  v = 0.0;
  for (int k = 0; k < TH / 64; ++k) {
    v += shd[k];
    m = max(m, shi[k]);
  }
}

// Cost in steps of one row slice of unit row = (b * Hkv + h) * nbmax + I, or
// kNoCost without queries.
__device__ __forceinline__ uint32_t unit_cost(const Problem& p, int cnt, int I, int b) {
  const int Lq = p.cu[b + 1] - p.cu[b], Lk = p.cuk[b + 1] - p.cuk[b];
  if (I * p.qtile >= Lq) return kNoCost;
  const int Ia = (Lk - Lq + min(Lq, (I + 1) * p.qtile) - 1) / kBlock;
  const int pruned = p.corr ? max(0, Ia + 1 - cnt) : 0;   // at most, below the last block
  return (uint32_t)(2 * cnt + (pruned + 63) / 64 + kItemSteps);
}

// Lanes of the wave that are `on` and hold the same key (6 bits) as this one.
__device__ __forceinline__ uint64_t match_key(int key, bool on) {
  uint64_t m = __ballot(on);
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const uint64_t b = __ballot((key >> i) & 1);
    m &= (key >> i) & 1 ? b : ~b;
  }
  return m;
}

// Smallest step budget of the cost-balanced mode for a call of `units` units.
__host__ __device__ __forceinline__ int min_split_steps(const Problem& p, int64_t units, const Plan& plan) {
  return !p.fp8 && units * plan.wpu * 16 <= plan.resident ? kMinSplitStepsFewBf16 : kMinSplitSteps;
}

// Units are indexed in attention order q = (nbmax - 1 - I) * nbh + bh, unit row
// bh * nbmax + I. Workgroup g of gridDim.x writes the entries of units
// [g * chunk, (g + 1) * chunk).
template <int TH>
__global__ __launch_bounds__(TH) void plan_kernel(Problem p, KeptLists kl, Plan plan,
                                                            int wpu) {
  constexpr int kWaves = TH / 64;
  __shared__ double shd[kWaves];
  __shared__ int shi[kWaves];
  __shared__ uint16_t sc[kCostCache];
  // items per class of unsplit and of split units: all of them, and those of
  // earlier workgroups' units; a class's table entries are those of its split
  // units, then the unsplit ones in attention order
  __shared__ int hist[4 * kClasses];
  __shared__ int pos[2 * kClasses];    // next entries of a class for this workgroup: unsplit, split
  __shared__ int wtot[kWaves][kClasses];
  __shared__ int next[2];              // next partial slot and split-list entry
  const int tid = threadIdx.x;
  const int nbh = p.batch * p.hkv;
  const int R = nbh * p.nbmax;
  const int chunk = (R + (int)gridDim.x - 1) / (int)gridDim.x;
  const int q0 = min(R, (int)blockIdx.x * chunk), q1 = min(R, q0 + chunk);
  const bool in_lds = R <= kCostCache;
  auto cost_of = [&](int q) -> uint32_t {
    if (in_lds) return sc[q];
    const int I = p.nbmax - 1 - q / nbh, bh = q % nbh;
    return unit_cost(p, kl.cnt[bh * p.nbmax + I], I, bh / p.hkv);
  };

  // costs, read in the order of the rows (coalesced), four rows in flight
  double tot = 0.0;
  int mx = 0;
  for (int r0 = tid; r0 < R; r0 += 4 * TH) {
    int cnt[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = r0 + j * TH;
      cnt[j] = row < R ? kl.cnt[row] : 0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = r0 + j * TH;
      if (row >= R) break;
      const int bh = row / p.nbmax, I = row - bh * p.nbmax;
      const uint32_t c = unit_cost(p, cnt[j], I, bh / p.hkv);
      if (c != kNoCost) {
        tot += (double)c * wpu;
        mx = max(mx, (int)c);
      }
      if (in_lds) sc[(p.nbmax - 1 - I) * nbh + bh] = (uint16_t)c;
    }
  }
  if (tid < 4 * kClasses) hist[tid] = 0;
  if (tid < 2) next[tid] = 0;
  block_sum_max<TH>(tot, mx, shd, shi);   // (its barriers also publish sc)

  // one resident workgroup's share of the call's steps
  const double share = tot / (double)max(1, plan.resident);
  const bool sorted = plan.resident_per_cu == 1 && (double)mx > (p.fp8 ? kSortAboveFp8 : kSortAboveBf16) * share;

  // step budget of the cost-balanced mode
  int S = 0;
  if (p.splits == 0) {
    S = max(min_split_steps(p, R, plan), (int)ceil(share));
    while (S < mx) {   // grow S until the parts fit the partial-output slots
      double need = 0.0;
      int none = 0;
      for (int q = tid; q < R; q += TH) {
        const uint32_t c = cost_of(q);
        if (c != kNoCost && (int)c > S) need += min(kMaxRowSplits, ((int)c + S - 1) / S);
      }
      block_sum_max<TH>(need, none, shd, shi);
      if (need <= (double)plan.cap_slots) break;
      S = max(S + max(1, S / 4), (int)((double)S * need / (double)max(1, plan.cap_slots)));
    }
  }
  auto parts = [&](uint32_t c) -> int {
    if (c == kNoCost) return 0;
    if (p.splits > 0) return p.splits;
    return (int)c > S ? min(kMaxRowSplits, ((int)c + S - 1) / S) : 1;
  };
  // class of a unit's parts: linear in their cost, 0 the heaviest
  const int top = p.splits > 0 ? (mx + p.splits - 1) / p.splits
                               : max(min(mx, S), (mx + kMaxRowSplits - 1) / kMaxRowSplits);
  auto class_of = [&](uint32_t c, int U) -> int {
    if (!sorted) return 0;
    const int pc = min(top, ((int)c + U - 1) / U);
    return kClasses - 1 - (int)((uint32_t)pc * kClasses / (uint32_t)(top + 1));
  };

  // items per class, of all units and of those before q0; partial slots and
  // split units before q0 (units of one part by ballots, the others one by one)
  for (int qb = 0; qb < R; qb += TH) {
    const int q = qb + tid;
    const uint32_t c = q < R ? cost_of(q) : kNoCost;
    const int U = parts(c);
    const int cl = U > 0 ? class_of(c, U) : 0;
    const bool before = q < q0;
    const uint64_t m = match_key(cl | (before ? kClasses : 0), U == 1);
    if (U == 1 && (m & ((1ull << (tid & 63)) - 1ull)) == 0) {
      const int n = __popcll(m) * wpu;
      atomicAdd(&hist[cl], n);
      if (before) atomicAdd(&hist[kClasses + cl], n);
    } else if (U > 1) {
      atomicAdd(&hist[2 * kClasses + cl], U * wpu);
      if (before) {
        atomicAdd(&hist[3 * kClasses + cl], U * wpu);
        atomicAdd(&next[0], U);
        atomicAdd(&next[1], 1);
      }
    }
  }
  __syncthreads();
  if (tid < kClasses) {
    int at = 0;
    for (int k = 0; k < tid; ++k) at += hist[k] + hist[2 * kClasses + k];
    pos[kClasses + tid] = at + hist[3 * kClasses + tid];
    pos[tid] = at + hist[2 * kClasses + tid] + hist[kClasses + tid];
  }
  __syncthreads();

  // entries of this workgroup's units; an unsplit unit's rank is that among
  // the lower lanes of the wave, then over the waves in turn
  const int lane = tid & 63, w = tid >> 6;
  for (int qb = q0; qb < q1; qb += TH) {
    const int q = qb + tid;
    const uint32_t c = q < q1 ? cost_of(q) : kNoCost;
    const int U = parts(c);
    const int cl = U > 0 ? class_of(c, U) : 0;
    const uint64_t m = match_key(cl, U == 1);
    const int rank = __popcll(m & ((1ull << lane) - 1ull));
    if (tid < kClasses) {
#pragma unroll
      for (int v = 0; v < kWaves; ++v) wtot[v][tid] = 0;
    }
    __syncthreads();
    if (U == 1 && (m >> lane) == 1) wtot[w][cl] = (rank + 1) * wpu;   // the class's last lane
    __syncthreads();
    if (tid < kClasses) {
      int at = pos[tid];
#pragma unroll
      for (int v = 0; v < kWaves; ++v) {
        const int n = wtot[v][tid];
        wtot[v][tid] = at;
        at += n;
      }
      pos[tid] = at;
    }
    __syncthreads();
    if (q < q1) {
      const int row = (q % nbh) * p.nbmax + (p.nbmax - 1 - q / nbh);
      int slot = -1, at = wtot[w][cl] + rank * wpu;
      if (U > 1) {
        at = atomicAdd(&pos[kClasses + cl], U * wpu);
        slot = atomicAdd(&next[0], U);
        plan.splitrows[atomicAdd(&next[1], 1)] = row;
      }
      plan.rowinfo[row] = U > 0 ? make_int2(U, slot) : make_int2(-1, -1);
      for (int k = 0; k < U * wpu; ++k) plan.items[at + k] = make_int4(q, k, U, slot);
    }
    __syncthreads();
  }
  // (the last workgroup's running totals end at the call's)
  __syncthreads();
  if (blockIdx.x == gridDim.x - 1 && tid == 0) {
    int ti = 0;
    for (int k = 0; k < kClasses; ++k) ti += hist[k] + hist[2 * kClasses + k];
    plan.counts[0] = 0;
    plan.counts[1] = ti;
    plan.counts[2] = next[1];
  }
}

template <int FP8>
__global__ __launch_bounds__(256) void combine_kernel(Problem p, Plan plan,
                                                      uint16_t* __restrict__ out,
                                                      float* __restrict__ lse) {
  const int G = p.g, rpu = G * p.qtile, groups = rpu / 8;
  const int work = plan.counts[2] * groups;
  const int lane = threadIdx.x & 31, sub = threadIdx.x >> 5;
  const int c = lane * 4;
  const float off = FP8 ? 8.f : 0.f;
#pragma unroll 1
  for (int wk = blockIdx.x; wk < work; wk += gridDim.x) {
    const int sr = wk / groups, grp = wk - sr * groups;
    const int row = plan.splitrows[sr];
    const int2 ri = plan.rowinfo[row];
    const int U = ri.x, slot0 = ri.y;
    const int I = row % p.nbmax, bh = row / p.nbmax;
    const int b = bh / p.hkv, h = bh % p.hkv;
    const int pr = grp * 8 + sub;              // packed row of this half-wave
    const int pos = I * p.qtile + pr / G;
    if (pos >= p.cu[b + 1] - p.cu[b]) continue;
    // lane u holds {m, l} of parts u and u + 32
    float m[2], l[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      m[k] = -INFINITY;
      l[k] = 0.f;
      if (lane + 32 * k < U) {
        const float2 ml =
            *(const float2*)(plan.part_ml + 2 * ((int64_t)(slot0 + lane + 32 * k) * rpu + pr));
        m[k] = ml.x;
        l[k] = ml.y;
      }
    }
    float M = fmaxf(m[0], m[1]);
    for (int o = 16; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 32));
    float wgt[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) wgt[k] = m[k] == -INFINITY ? 0.f : fast_exp2(m[k] - M);
    float lt = wgt[0] * l[0] + wgt[1] * l[1];
    for (int o = 16; o > 0; o >>= 1) lt += __shfl_xor(lt, o, 32);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int u0 = 0; u0 < U; u0 += 4) {   // four parts' loads in flight at a time
      float wu[4];
      float4 o[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int u = u0 + k;
        wu[k] = __shfl(u < 32 ? wgt[0] : wgt[1], u & 31, 32);
        o[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (u < U && wu[k] != 0.f)
          o[k] = *(const float4*)(plan.part_o + ((int64_t)(slot0 + u) * rpu + pr) * kHeadDim + c);
        else
          wu[k] = 0.f;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        acc.x = fmaf(wu[k], o[k].x, acc.x);
        acc.y = fmaf(wu[k], o[k].y, acc.y);
        acc.z = fmaf(wu[k], o[k].z, acc.z);
        acc.w = fmaf(wu[k], o[k].w, acc.w);
      }
    }
    const float inv = (FP8 ? p.v_scale[h] : 1.f) / lt;
    const int hq = h * G + pr % G;
    const int64_t t = (int64_t)p.cu[b] + pos;
    uint2 v;
    v.x = pack_bf16x2(acc.x * inv, acc.y * inv);
    v.y = pack_bf16x2(acc.z * inv, acc.w * inv);
    *(uint2*)(out + (t * p.hq + hq) * kHeadDim + c) = v;
    if (lse && lane == 0) lse[t * p.hq + hq] = (M + fast_log2(lt) - off) * kLn2;
  }
}

}  // namespace

// Compute units of the current device, queried once per device; the cache is
// atomic so that calls from several host threads are well defined (each may
// query and store the same value).
int device_compute_units() {
  static std::atomic<int> cus[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

hipError_t launch_plan(const Problem& p, const KeptLists& kl, const Plan& plan, hipStream_t s) {
  if (p.batch == 0 || p.nbmax == 0) return hipSuccess;
  const int64_t units = (int64_t)p.batch * p.hkv * p.nbmax;
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(kPlanGroups, units / kPlanUnits));
  const int wpu = plan.wpu;
  if (units <= kPlanFewUnits)
    plan_kernel<kPlanThreadsFew><<<grid, kPlanThreadsFew, 0, s>>>(p, kl, plan, wpu);
  else
    plan_kernel<kPlanThreads><<<grid, kPlanThreads, 0, s>>>(p, kl, plan, wpu);
  return hipGetLastError();
}

hipError_t launch_combine(const Problem& p, const Plan& plan, void* out, float* lse,
                          hipStream_t s) {
  if (p.batch == 0 || p.nbmax == 0 || plan.cap_slots == 0) return hipSuccess;
  // Short sequences: even a unit that keeps every key block stays within the
  // smallest step budget, so nothing is split (4 us of a 43 us call).
  const int64_t units = (int64_t)p.batch * p.hkv * p.nbmax;
  if (p.splits == 0 && 2 * p.nbk + kItemSteps <= min_split_steps(p, units, plan)) return hipSuccess;
  const int64_t bound = (int64_t)(plan.cap_slots / 2) * (p.g * p.qtile / 8);
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(bound, 1024));
  if (p.fp8)
    combine_kernel<1><<<grid, 256, 0, s>>>(p, plan, (uint16_t*)out, lse);
  else
    combine_kernel<0><<<grid, 256, 0, s>>>(p, plan, (uint16_t*)out, lse);
  return hipGetLastError();
}

}  // namespace fp2
