// Block means of K and V (Sec. 3.2, the pooled statistics kbar_J, vbar_J of
// Eq. correction; the block means of Algorithm 1). HBM-bound: every K/V byte of the
// sequence is read once with 16-byte loads through the page table.
//
// A workgroup of 256 threads takes one (key block J, KV head h, sequence b) of
// the sequence's KV tokens (a prefix included) at a time: one in all without a
// means cache, the uncached ones in turn with it (pool_cached_kernel).
//  - bf16: thread (row group rg = tid/16, column chunk c = tid%16) sums tokens
//    rg, rg+16, ... of the block for columns 8c..8c+7 in fp64. Every bf16
//    value is exact in fp64 and so are the partial sums of realistic data, so
//    the mean does not depend on the summation order.
//  - fp8: each e4m3 value is an exact multiple of 2^-9 (the hardware decode
//    v_cvt_pk_f32_fp8 is exact); per-thread sums of 4 rows are exact in fp32,
//    the block sums exact 32-bit integers in units of 2^-9, and the mean is
//    (sum * 2^-9 * scale) / count in fp64 (the product is exact, the
//    division rounds once).
// The rounded key mean khat (bf16, one rounding from fp64) is the scoring key
// of Eq. fused_score and the surrogate key of the correction; vbar is the
// value mean in bf16. For fp8 inputs the correction runs on the matrix cores
// in fp8 like the kept keys (the pooled statistics quantized as Sec. 4 does
// under fp8): the kernel also writes the e4m3 code means e4m3(khat / k_scale)
// and e4m3(vbar / v_scale), derived from the bf16 means so that blocks taken
// from a means cache give the same codes. With a caller's means cache (chunked
// prefill), complete blocks it already holds are copied from it (512 bytes per
// block and head instead of the block's K/V), and every block pooled here is
// written to it.
#include <algorithm>

#include "kernels.h"

namespace fp2 {

namespace {

constexpr int kThreads = 256;

// Element offset of (key block J of sequence b, KV head h) in the caller's
// means cache.
__device__ __forceinline__ int64_t cache_offset(const Problem& p, const MeansCache& mc, int b,
                                                int J, int h) {
  int64_t slot;
  if (p.pm.page == 0) {
    slot = (int64_t)b * p.nbk + J;
  } else {
    const int t = J * kBlock;
    const int pg = p.pm.shift >= 0 ? t >> p.pm.shift : t / p.pm.page;
    const int off = t - pg * p.pm.page;
    slot = (int64_t)p.pm.table[(int64_t)b * p.pm.stride + pg] * mc.per_page + off / kBlock;
  }
  return (slot * p.hkv + h) * kHeadDim;
}

// e4m3 code of a bf16 mean (|mean / scale| <= 448).
__device__ __forceinline__ uint32_t code_of(uint16_t mean, float scale) {
  const float c = __uint_as_float((uint32_t)mean << 16) / scale;
  return __builtin_amdgcn_cvt_pk_fp8_f32(fminf(fmaxf(c, -448.f), 448.f), 0.f, 0, false) & 0xFF;
}

// Leading blocks of sequence b (L KV tokens) that the caller's cache holds.
__device__ __forceinline__ int cached_blocks(const MeansCache& mc, int b, int L) {
  return max(0, min(mc.pooled[b], L / kBlock));
}

// Means of one block (zero past the sequence) by a workgroup; also to the
// block's slot of a caller's cache.
template <int FP8>
__device__ __forceinline__ void pool_block(const Problem& p, const Pooled& out, const MeansCache& mc,
                                           int J, int h, int b, int tid) {
  const int64_t tok0 = p.cuk[b];
  const int L = p.cuk[b + 1] - (int)tok0;     // KV tokens, a prefix included
  const int64_t obase = (((int64_t)b * p.hkv + h) * p.nbk + J) * kHeadDim;
  const int n = (L + kBlock - 1) / kBlock;
  // fp8: the e4m3 code means, from the bf16 means
  auto store8 = [&](uint16_t kh, uint16_t vb) {
    if (FP8 && out.khat8) {
      out.khat8[obase + tid] = (uint8_t)code_of(kh, p.k_scale[h]);
      out.vbar8[obase + tid] = (uint8_t)code_of(vb, p.v_scale[h]);
    }
  };
  if (J >= n) {
    if (tid < kHeadDim) {
      out.khat[obase + tid] = 0;
      out.vbar[obase + tid] = 0;
      store8(0, 0);
    }
    return;
  }
  const int64_t cbase = mc.khat ? cache_offset(p, mc, b, J, h) : 0;
  // the means go to the workspace and, with a cache, to the block's slot
  auto store = [&](uint16_t kh, uint16_t vb) {
    out.khat[obase + tid] = kh;
    out.vbar[obase + tid] = vb;
    store8(kh, vb);
    if (mc.khat) {
      mc.khat[cbase + tid] = kh;
      mc.vbar[cbase + tid] = vb;
    }
  };
  const int cnt = min(kBlock, L - J * kBlock);

  if constexpr (!FP8) {
    __shared__ double redk[16][kHeadDim];
    __shared__ double redv[16][kHeadDim];
    const int c = tid & 15, rg = tid >> 4;
    double ak[8], av[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) ak[i] = av[i] = 0.0;
    const uint16_t* K = (const uint16_t*)p.k;
    const uint16_t* V = (const uint16_t*)p.v;
    // all 2 x 8 loads of this thread in flight before the first sum; rows
    // past the block read nothing and add zero
    uint4 kv[8], vv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = rg + 16 * i;
      kv[i] = vv[i] = make_uint4(0, 0, 0, 0);
      if (r < cnt) {
        const int64_t off = (slot_of(p.pm, b, tok0, J * kBlock + r) * p.hkv + h) * kHeadDim + c * 8;
        kv[i] = *(const uint4*)(K + off);
        vv[i] = *(const uint4*)(V + off);
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const uint32_t kw[4] = {kv[r].x, kv[r].y, kv[r].z, kv[r].w};
      const uint32_t vw[4] = {vv[r].x, vv[r].y, vv[r].z, vv[r].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        ak[2 * i] += (double)__uint_as_float(kw[i] << 16);
        ak[2 * i + 1] += (double)__uint_as_float(kw[i] & 0xFFFF0000u);
        av[2 * i] += (double)__uint_as_float(vw[i] << 16);
        av[2 * i + 1] += (double)__uint_as_float(vw[i] & 0xFFFF0000u);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      redk[rg][c * 8 + i] = ak[i];
      redv[rg][c * 8 + i] = av[i];
    }
    __syncthreads();
    if (tid < kHeadDim) {
      double sk = 0.0, sv = 0.0;
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        sk += redk[g][tid];
        sv += redv[g][tid];
      }
      store(f64_to_bf16(sk / (double)cnt), f64_to_bf16(sv / (double)cnt));
    }
  } else {
    // 8 threads per token row (16 codes each), 32 row groups.
    const int c = tid & 7, rg = tid >> 3;
    const uint8_t* K = (const uint8_t*)p.k;
    const uint8_t* V = (const uint8_t*)p.v;
    uint4 kv[4], vv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = rg + 32 * i;
      kv[i] = vv[i] = make_uint4(0, 0, 0, 0);
      if (r < cnt) {
        const int64_t off = (slot_of(p.pm, b, tok0, J * kBlock + r) * p.hkv + h) * kHeadDim + c * 16;
        kv[i] = *(const uint4*)(K + off);
        vv[i] = *(const uint4*)(V + off);
      }
    }
    // Codes decoded by the hardware (v_cvt_pk_f32_fp8, exact) and summed in
    // fp32 over the thread's 4 rows: every e4m3 value is a multiple of 2^-9
    // below 448 in magnitude, so a sum of 4 needs at most 20 significant
    // bits and is exact; times 512 it is an exact integer.
    float fk[16], fv[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) fk[i] = fv[i] = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const uint32_t kw[4] = {kv[r].x, kv[r].y, kv[r].z, kv[r].w};
      const uint32_t vw[4] = {vv[r].x, vv[r].y, vv[r].z, vv[r].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x2_t k0 = __builtin_amdgcn_cvt_pk_f32_fp8((int)kw[q], false);
        const f32x2_t k1 = __builtin_amdgcn_cvt_pk_f32_fp8((int)kw[q], true);
        const f32x2_t v0 = __builtin_amdgcn_cvt_pk_f32_fp8((int)vw[q], false);
        const f32x2_t v1 = __builtin_amdgcn_cvt_pk_f32_fp8((int)vw[q], true);
        fk[4 * q] += k0.x;
        fk[4 * q + 1] += k0.y;
        fk[4 * q + 2] += k1.x;
        fk[4 * q + 3] += k1.y;
        fv[4 * q] += v0.x;
        fv[4 * q + 1] += v0.y;
        fv[4 * q + 2] += v1.x;
        fv[4 * q + 3] += v1.y;
      }
    }
    int ak[16], av[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      ak[i] = (int)(fk[i] * 512.f);
      av[i] = (int)(fv[i] * 512.f);
    }
    // integer sums (exact): over the wave's 8 row groups with lane
    // exchanges, then over the 4 waves through LDS (4 KiB, so LDS does not
    // bound the workgroups per CU)
    __shared__ int redki[4][kHeadDim];
    __shared__ int redvi[4][kHeadDim];
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int o = 8; o < 64; o <<= 1) {
        ak[i] += __shfl_xor(ak[i], o, 64);
        av[i] += __shfl_xor(av[i], o, 64);
      }
    const int w = tid >> 6;
    if ((tid & 63) < 8) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        redki[w][c * 16 + i] = ak[i];
        redvi[w][c * 16 + i] = av[i];
      }
    }
    __syncthreads();
    if (tid < kHeadDim) {
      const int sk = (redki[0][tid] + redki[1][tid]) + (redki[2][tid] + redki[3][tid]);
      const int sv = (redvi[0][tid] + redvi[1][tid]) + (redvi[2][tid] + redvi[3][tid]);
      double ks = (double)p.k_scale[h], vs = (double)p.v_scale[h];
      store(f64_to_bf16(((double)sk * 0x1p-9 * ks) / (double)cnt),
            f64_to_bf16(((double)sv * 0x1p-9 * vs) / (double)cnt));
    }
  }
}

template <int FP8>
__global__ __launch_bounds__(kThreads) void pool_kernel(Problem p, Pooled out) {
  pool_block<FP8>(p, out, MeansCache{nullptr, nullptr, nullptr, 0}, blockIdx.x, blockIdx.y, blockIdx.z,
                  threadIdx.x);
}

// With a caller's cache: the first `poolers` workgroups of a KV head share the
// uncached blocks of all sequences, counted on the device, since the host knows
// neither how many the cache holds nor in which sequence they are missing; the
// others copy the cached means and zero the blocks past a sequence, kCopyBlocks
// blocks each with 16-byte accesses. The poolers fill the chip once over all
// heads (their registers admit kPoolersBf16 / kPoolersFp8 on a compute unit) and
// come first: the last workgroups of a grid start some 10 us after the first.
// One workgroup per block, which for a short extend was almost only copies of 512
// bytes, took 14.3 us for 128 fp8 tokens after 131K; this takes 9.8 (an 8K bf16
// chunk after 56K 14.3 -> 13.4, four fp8 extends 31 -> 22). Prefixes the cache does
// not hold: 57K bf16 42 -> 39 us, 131K fp8 59 -> 68, 100K of one of 16 sequences
// 138 -> 104, four fp8 extends 137 -> 146; pooled by one workgroup per query block,
// as if every prefix were cached, these took 1190, 2700, 2730 and 2730.
constexpr int kCopyBlocks = 16;
constexpr int kPoolersBf16 = 4, kPoolersFp8 = 5;

template <int FP8>
__global__ __launch_bounds__(kThreads) void pool_cached_kernel(Problem p, Pooled out, MeansCache mc,
                                                               int poolers, int copiers) {
  const int h = blockIdx.x % p.hkv, i = blockIdx.x / p.hkv, tid = threadIdx.x;
  if (i >= poolers) {
    const int tiles = (p.nbk + kCopyBlocks - 1) / kCopyBlocks;   // per sequence
    for (int64_t k = i - poolers; k < (int64_t)tiles * p.batch; k += copiers) {
      const int b = (int)(k / tiles), J = (int)(k - (int64_t)b * tiles) * kCopyBlocks + tid / 16;
      const int c = tid % 16 * 8;
      const int L = p.cuk[b + 1] - p.cuk[b];
      const int held = cached_blocks(mc, b, L), n = (L + kBlock - 1) / kBlock;
      if (J >= p.nbk || (J >= held && J < n)) continue;
      const int64_t ob = (((int64_t)b * p.hkv + h) * p.nbk + J) * kHeadDim + c;
      uint4 kh = make_uint4(0, 0, 0, 0), vb = kh;   // past the sequence
      if (J < held) {
        const int64_t cb = cache_offset(p, mc, b, J, h) + c;
        kh = *(const uint4*)(mc.khat + cb);
        vb = *(const uint4*)(mc.vbar + cb);
      }
      *(uint4*)(out.khat + ob) = kh;
      *(uint4*)(out.vbar + ob) = vb;
      if (FP8 && out.khat8) {
        auto codes = [](const uint4& m, float scale) -> uint2 {
          const uint32_t w[4] = {m.x, m.y, m.z, m.w};
          uint32_t r[2];
#pragma unroll
          for (int j = 0; j < 2; ++j)
            r[j] = code_of((uint16_t)w[2 * j], scale) | code_of((uint16_t)(w[2 * j] >> 16), scale) << 8 |
                   code_of((uint16_t)w[2 * j + 1], scale) << 16 |
                   code_of((uint16_t)(w[2 * j + 1] >> 16), scale) << 24;
          return make_uint2(r[0], r[1]);
        };
        *(uint2*)(out.khat8 + ob) = codes(kh, p.k_scale[h]);
        *(uint2*)(out.vbar8 + ob) = codes(vb, p.v_scale[h]);
      }
    }
    return;
  }
  // this workgroup's share of the head's uncached blocks, sequence after
  // sequence; lane l of every wave knows sequence b0 + l
  int t = i, at = 0;
  for (int b0 = 0; b0 < p.batch; b0 += 64) {
    const int lane = tid & 63, bl = b0 + lane;
    int held = 0, fresh = 0;
    if (bl < p.batch) {
      const int L = p.cuk[bl + 1] - p.cuk[bl];
      held = cached_blocks(mc, bl, L);
      fresh = max(0, min(p.nbk, (L + kBlock - 1) / kBlock) - held);
    }
    int upto = fresh;   // uncached blocks of the sequences b0 .. bl
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(upto, o, 64);
      if (lane >= o) upto += v;
    }
    const int first = held - (upto - fresh);   // block of a sequence's share 0 of b0's
    const int end = at + __builtin_amdgcn_readlane(upto, 63);
    for (; t < end; t += poolers) {
      const int l = __ffsll((unsigned long long)__ballot(at + upto > t)) - 1;
      const int J = t - at + __builtin_amdgcn_readlane(first, l);
      int tb = tid;   // opaque: what pool_block derives from it is not held across the loop
      asm volatile("" : "+v"(tb));
      pool_block<FP8>(p, out, mc, J, h, b0 + l, tb);
      __syncthreads();   // the reduction buffers are free again
    }
    at = end;
  }
}

}  // namespace

hipError_t launch_pool(const Problem& p, Pooled out, hipStream_t s, const MeansCache& cache) {
  if (p.batch == 0 || p.nbk == 0) return hipSuccess;
  if (cache.khat) {
    const int64_t blocks = (int64_t)p.nbk * p.batch;
    const int64_t tiles = (int64_t)((p.nbk + kCopyBlocks - 1) / kCopyBlocks) * p.batch;
    const int fill = ((p.fp8 ? kPoolersFp8 : kPoolersBf16) * device_compute_units() + p.hkv - 1) / p.hkv;
    const int poolers = (int)std::min<int64_t>(blocks, std::max(1, fill));
    const int copiers = (int)std::min<int64_t>(tiles, (1 << 22) / p.hkv);   // within the largest grid
    const unsigned grid = (unsigned)(poolers + copiers) * p.hkv;
    if (p.fp8)
      pool_cached_kernel<1><<<grid, kThreads, 0, s>>>(p, out, cache, poolers, copiers);
    else
      pool_cached_kernel<0><<<grid, kThreads, 0, s>>>(p, out, cache, poolers, copiers);
    return hipGetLastError();
  }
  const dim3 grid(p.nbk, p.hkv, p.batch);
  if (p.fp8)
    pool_kernel<1><<<grid, kThreads, 0, s>>>(p, out);
  else
    pool_kernel<0><<<grid, kThreads, 0, s>>>(p, out);
  return hipGetLastError();
}

}  // namespace fp2
