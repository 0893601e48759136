// Combine (weighted sum over the top-k expert outputs in token order) and the kernels of the deduplicating
// high-throughput mode: dedup, per-expert index list, partial reduce per group.
#include <cmath>

#include "ep_device.h"

namespace ep {

// ---------------------------------------------------------------- combine
// out[t, 8 channels] = bf16( sum_k w[t,k] * y[row_k, 8 channels] ): per 16-byte
// column slice, K independent 16-byte loads are in flight per lane, then the
// fp32 fused multiply-add chain runs in ascending k from +0, and the result is
// rounded once (nearest even) to bf16.  Rows and weights are wave-uniform.
EP_DEV unsigned pack_bf16_rne(float a, float b) {
  unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
  ua = (ua + 0x7FFFu + ((ua >> 16) & 1u)) >> 16;
  ub = (ub + 0x7FFFu + ((ub >> 16) & 1u)) & 0xFFFF0000u;
  return ua | ub;
}

EP_DEV void fma8(float (&acc)[8], float w, const u32x4 &v) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    acc[2 * j] = __builtin_fmaf(w, bf16_lo(v[j]), acc[2 * j]);
    acc[2 * j + 1] = __builtin_fmaf(w, bf16_hi(v[j]), acc[2 * j + 1]);
  }
}

// The slices of one wave, one after the other: K loads in flight, the chain in ascending k, the packed
// result kept in registers; the stores of all slices leave together at the end, so that a wave's writes
// do not trickle into its reads.  STREAM: non-temporal loads (rows that no cache is expected to hold).  SKIP: masked entries load
// nothing, else a row that is loaded anyway.
template <int VPL, int KT, bool STREAM, bool SKIP>
EP_DEV void combine_slices(const u32x4 *y, u32x4 *out, const int (&rows)[KT], const float (&ws)[KT], int safe, int nvec,
                           int v0) {
  u32x4 res[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i)
    if (v0 + i * 64 < nvec) {
      u32x4 ld[KT];
#pragma unroll
      for (int k = 0; k < KT; ++k) {
        if (SKIP && rows[k] < 0) continue;
        const u32x4 *p = y + (size_t)(rows[k] >= 0 ? rows[k] : safe) * nvec + v0 + i * 64;
        ld[k] = STREAM ? __builtin_nontemporal_load(p) : *p;
      }
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KT; ++k)
        if (rows[k] >= 0) fma8(acc, ws[k], ld[k]);
      res[i] = u32x4{pack_bf16_rne(acc[0], acc[1]), pack_bf16_rne(acc[2], acc[3]), pack_bf16_rne(acc[4], acc[5]),
                     pack_bf16_rne(acc[6], acc[7])};
    }
#pragma unroll
  for (int i = 0; i < VPL; ++i)
    if (v0 + i * 64 < nvec) __builtin_nontemporal_store(res[i], out + v0 + i * 64);
}

template <int VPL, int KT>
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a) {
  const int lane = lane_id();
  const unsigned item = blockIdx.x * (unsigned)a.group_waves + wave_id();
  const int t_launch = (int)(item / (unsigned)a.parts), part = (int)(item % (unsigned)a.parts);
  if (t_launch >= a.T) return;
  // With fresh rows the grid starts at the end of the token range where they are (the last tokens,
  // or the first ones when the kernel that wrote them went backwards) and takes the newest first:
  // the rows written last are read before the rest of the traffic pushes them out of the
  // memory-side cache.
  const int n_fresh = a.T - a.fresh_from;
  const int t = (n_fresh > 0 && !a.fresh_head) ? a.T - 1 - t_launch : t_launch;
  const bool fresh = a.fresh_head ? t < n_fresh : t >= a.fresh_from;
  const int K = KT > 0 ? KT : a.K;
  int row = -1;
  float wt = 0.0f;
  if (lane < K) {
    row = a.dst_row[(size_t)t * K + lane];
    wt = a.w[(size_t)t * K + lane];
    if (row < -1 || row >= a.y_rows) {
      dev_set_error(a.error, EP_EBOUNDS);
      row = -1;
    }
  }
  const unsigned long long vmask = __ballot(row >= 0);
  const int nvec = a.H >> 3;
  const int v0 = part * VPL * 64 + lane;
  u32x4 *out = (u32x4 *)a.out + (size_t)t * nvec;
  if (vmask == 0) {  // every k masked: +0
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (v0 + i * 64 < nvec) out[v0 + i * 64] = u32x4{0, 0, 0, 0};
    return;
  }
  const u32x4 *y = (const u32x4 *)a.y;
  if constexpr (KT > 0) {
    const int safe = __builtin_amdgcn_readlane(row, __builtin_ctzll(vmask));
    int rows[KT];
    float ws[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      rows[k] = __builtin_amdgcn_readlane(row, k);
      ws[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), k));
    }
    // (wave-uniform; two instances so that each keeps its own kind of load)
    if (fresh) {
      combine_slices<VPL, KT, false, false>(y, out, rows, ws, safe, nvec, v0);
      // (keeps the optimiser from folding the two instances into one, which drops the streaming hint of the other)
      asm volatile("" ::: "memory");
    } else {
      combine_slices<VPL, KT, true, false>(y, out, rows, ws, safe, nvec, v0);
    }
  } else {
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (v0 + i * 64 < nvec) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < K; ++k) {
          const int r = __builtin_amdgcn_readlane(row, k);
          const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), k));
          if (r >= 0) fma8(acc, w, __builtin_nontemporal_load(y + (size_t)r * nvec + v0 + i * 64));
        }
        u32x4 o = {pack_bf16_rne(acc[0], acc[1]), pack_bf16_rne(acc[2], acc[3]),
                   pack_bf16_rne(acc[4], acc[5]), pack_bf16_rne(acc[6], acc[7])};
        __builtin_nontemporal_store(o, out + v0 + i * 64);
      }
  }
}

// The same with one slice per wave and loads for the entries that have a row only, for rows that no cache is expected to hold.
template <int KT>
__global__ __launch_bounds__(256) void combine_slice_kernel(CombineArgs a) {
  const int lane = lane_id();
  const unsigned item = blockIdx.x * (unsigned)a.group_waves + wave_id();
  const int t = (int)(item / (unsigned)a.parts), part = (int)(item % (unsigned)a.parts);
  if (t >= a.T) return;
  int row = -1;
  float wt = 0.0f;
  if (lane < KT) {
    row = a.dst_row[(size_t)t * KT + lane];
    wt = a.w[(size_t)t * KT + lane];
    if (row < -1 || row >= a.y_rows) {
      dev_set_error(a.error, EP_EBOUNDS);
      row = -1;
    }
  }
  const int nvec = a.H >> 3;
  int rows[KT];
  float ws[KT];
#pragma unroll
  for (int k = 0; k < KT; ++k) {
    rows[k] = __builtin_amdgcn_readlane(row, k);
    ws[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), k));
  }
  combine_slices<1, KT, true, true>((const u32x4 *)a.y, (u32x4 *)a.out + (size_t)t * nvec, rows, ws, 0, nvec, part * 64 + lane);
}

// Dynamic LDS (not used) that lets about `waves` one-wave workgroups onto a compute unit: it has 160 KB, given out in pieces of
// 1280 bytes.
static size_t lds_for_waves(int waves) { return waves >= 32 ? 0 : 163840 / waves / 1280 * 1280; }

// Waves per workgroup of both reduces: one, but four where all fit onto the chip at once (32 on each of 256 compute units) and
// where a wave has little to do: top-3 and less, in the partial reduce top-4.  There the rate at which workgroups start is what
// counts.  One / four, us: combine of 512 tokens x 4096 top-4 5.3 / 4.6, top-6 6.3 / 5.8, top-8 7.6 / 7.1, top-12 12.3 / 11.8,
// 512 x 7168 top-8 11.9 / 11.7, but 1024 x 5120 (10240 waves) 16.6 / 17.0, 3000 x 7168 top-4 35.2 / 35.7; 3000 x 7168 top-2
// 22.6 / 22.5, with eight tenths masked 14.9 / 14.4, top-1 13.6 / 11.4; partial reduce of 512 x 4096 top-4 7.3 / 5.8, top-6 9.6
// / 7.8, top-8 12.5 / 11.7.
static int reduce_group_waves(long long items, bool few) { return items <= 8192 || few ? 4 : 1; }

// One slice (64 lanes x 16 bytes) per wave, one wave per workgroup, and no more of them on a compute unit than have 96 KB of
// rows on their way if no entry is masked.  The kernel is bound by the memory behind the L2, which about 84 KB of scattered
// reads per compute unit keep busy and which serves more of them in a worse order; but masked entries load nothing, and how
// many there are only the GPU knows: with 84 KB a table with three tenths of its entries masked leaves the memory idle.  A
// launch that does not fill the chip five times over has no such limit, nor have top-4 and less.  The combine alone, 10 / 12 /
// 14 / 16 / 20 / 32 waves per compute unit, and four waves per workgroup with a load for every entry, us:
//   top-8  3000 tokens x 7168 61.7 / 61.3 / 62.3 / 62.7 / 63.9 / 64.8, 66.2; a tenth masked 60.9 / 59.7 / 60.2 / 60.8 /
//          61.3 / 62.3, 63.0; three tenths 51.8 / 48.8 / 47.4 / 47.0 / 47.7 / 48.4, 50.2; half 43.7 / 39.7 / 37.1 / 35.7 / 35.1
//          / 35.6, 40.1; eight tenths 35.4 / 31.5 / 28.5 / 26.3 / 23.1 / 20.7, 31.2; 6000 x 4096 71.5 / 71.9 / 72.8 / 73.1 /
//          74.1 / 75.6, 77.1, half masked 49.9 / 45.2 / 42.3 / 40.6 / 39.9 / 40.5, 45.1; whole steps of 4096 x 7168 in chunks
//          with 12 and 14 waves 193.7 and 195.4
//   top-6  3000 x 7168, 14 / 16 / 18 / 20 / 32 waves 48.3 / 48.5 / 48.9 / 49.2 / 49.9, 51.5, half masked 32.5 / 30.8 /
//          29.6 / 28.6 / 28.1, 32.0; top-5, 16 / 20 / 24 / 32 waves 41.9 / 42.4 / 42.6 / 42.9, 44.3, half masked 29.3 / 27.0 /
//          26.3 / 25.7, 28.9; top-4, 20 / 24 / 32 waves 35.2 / 35.2 / 35.3, 36.4, half masked 24.3 / 23.3 / 22.6, 24.5
// Two slices per wave, at their best number of waves, take 1% longer, four 5%; a wave per token 2%.
// A handle with one expert per rank is how the second level of the hierarchical reduce comes here, whose entries are masked but
// for the first of each group: of K entries over G groups about G (1 - (1 - 1/G)^K) have a row, for which 100 KB is best.
// Deduplicated steps with 84 / 92 / 100 / 110 / 120 / 140 KB, us: 4096 x 7168 top-8 over 16 groups 321 / 322 / 322 / 326 / 326
// / 330, 8192 x 4096 369 / 369 / 369 / 372 / 372 / 375, over 8 groups 322 / 316 / 313 / 313 / 315 / 320, over 4 groups 271 /
// 271 / 266 / 266 / 266 / 266; 3001 x 8192 264 / 264 / 260 / 262 / 262 / 265, top-6 264 / 259 / 257 / 258 / 261 / 267.  (Such a
// handle with nothing masked gets 19 waves for top-8 over 8 ranks: 4096 x 7168 85.8 us, with 16 waves 83.2, four per workgroup
// with no limit 86.2.)
// (Top-9 and more go through a loop with one load in flight per wave: no limit.  Nor where rows of a dispatch that has just
// ended are read out of the memory-side cache.)
static int combine_waves(const CombineArgs &a) {
  if (a.K > 8 || a.fresh_from < a.T) return 32;
  if (a.groups) return (int)(100.0 / (a.groups * (1.0 - pow(1.0 - 1.0 / a.groups, a.K))));
  return a.K <= 4 ? 32 : 96 / a.K;
}
// (2, 4 and 7 slices per wave are for experiments, EP_COMBINE_VPL; anything else leaves one.)
static int tuned_combine_vpl(int forced) { return forced == 2 || forced == 4 || forced == 7 ? forced : 1; }

template <int VPL>
static void launch_combine_t(CombineArgs a, hipStream_t st, const LaunchTiming *tm) {
  const int nvec = a.H / 8;
  a.parts = (nvec + VPL * 64 - 1) / (VPL * 64);
  const long long items = (long long)a.T * a.parts;
  const int waves = combine_waves(a);
  const size_t lds = items >= 5ll * 256 * waves ? lds_for_waves(waves) : 0;  // (never with more than one wave per workgroup)
  a.group_waves = reduce_group_waves(items, a.K <= 3);
  const unsigned grid = (unsigned)((items + a.group_waves - 1) / a.group_waves);
  const dim3 block(64 * a.group_waves);
  void *ev0 = tm ? tm->start : nullptr, *ev1 = tm ? tm->stop : nullptr;
  if (VPL == 1 && a.K <= 8 && a.fresh_from == a.T) {
    switch (a.K) {
      case 1: launch_kernel(combine_slice_kernel<1>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      case 2: launch_kernel(combine_slice_kernel<2>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      case 3: launch_kernel(combine_slice_kernel<3>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      case 4: launch_kernel(combine_slice_kernel<4>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      case 5: launch_kernel(combine_slice_kernel<5>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      case 6: launch_kernel(combine_slice_kernel<6>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      case 7: launch_kernel(combine_slice_kernel<7>, dim3(grid), block, lds, st, ev0, ev1, a); break;
      default: launch_kernel(combine_slice_kernel<8>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    }
    return;
  }
  switch (a.K) {
    case 1: launch_kernel(combine_kernel<VPL, 1>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 2: launch_kernel(combine_kernel<VPL, 2>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 3: launch_kernel(combine_kernel<VPL, 3>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 4: launch_kernel(combine_kernel<VPL, 4>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 5: launch_kernel(combine_kernel<VPL, 5>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 6: launch_kernel(combine_kernel<VPL, 6>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 7: launch_kernel(combine_kernel<VPL, 7>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    case 8: launch_kernel(combine_kernel<VPL, 8>, dim3(grid), block, lds, st, ev0, ev1, a); break;
    default: launch_kernel(combine_kernel<VPL, 0>, dim3(grid), block, lds, st, ev0, ev1, a); break;
  }
}

int launch_combine(const CombineArgs &a, const Tunables &tune, void *stream, const LaunchTiming *timing) {
  hipStream_t st = (hipStream_t)stream;
  if (a.T <= 0) return 0;
  if ((a.H / 8 + 63) / 64 > 65535) return (int)hipErrorInvalidValue;
  switch (tuned_combine_vpl(tune.combine_vpl)) {
    case 2: launch_combine_t<2>(a, st, timing); break;
    case 4: launch_combine_t<4>(a, st, timing); break;
    case 7: launch_combine_t<7>(a, st, timing); break;
    default: launch_combine_t<1>(a, st, timing); break;
  }
  return (int)hipGetLastError();
}

// -------------------------------------------------- high-throughput mode
// Dedup: an entry keeps its group if no earlier entry of the token named it.  One thread per entry; the entries of the
// workgroup's tokens meet in LDS.  Bound by latency (a load, the look at up to K - 1 earlier entries, two stores):
// 4096 tokens top-8 4.7 us; one thread per token, walking its entries in global memory with two divisions for
// each pair, took 12.7 us.
__global__ __launch_bounds__(256) void dedup_kernel(DedupArgs a) {
  __shared__ int s_e[256];
  const int K = a.K, tid = threadIdx.x, tpb = 256 / K, k = tid % K;
  const int span = a.E_loc * a.ranks_per_group;  // experts of a group
  const long long n = a.n_tokens * K;
  for (long long i0 = (long long)blockIdx.x * tpb * K; i0 < n; i0 += (long long)gridDim.x * tpb * K) {
    const long long i = i0 + tid;
    const bool active = tid < tpb * K && i < n;
    const int e = active ? a.idx[i] : -1;
    s_e[tid] = e;
    __syncthreads();
    int g = -1, first = -1;
    if (e >= 0 && e < a.E) {
      const unsigned lo = (unsigned)e / (unsigned)span * (unsigned)span;
      const int *in = s_e + (tid - k);
      first = k;
      for (int j = k - 1; j >= 0; --j)
        if ((unsigned)in[j] - lo < (unsigned)span) first = j;
      if (first == k) g = (int)(lo / (unsigned)span);
    } else if (e != -1) {
      dev_set_error(a.error, EP_EBOUNDS);
    }
    if (active) {
      a.group_idx[i] = g;
      a.first_k[i] = first;
    }
    __syncthreads();
  }
}

int launch_dedup(const DedupArgs &a, void *stream) {
  if (a.n_tokens <= 0) return 0;
  const int tpb = 256 / a.K;
  const long long nblk = (a.n_tokens + tpb - 1) / tpb;
  hipLaunchKernelGGL(dedup_kernel, dim3((unsigned)(nblk < 65536 ? nblk : 65536)), dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

__global__ __launch_bounds__(256) void gather_index_kernel(GatherIndexArgs a) {
  const unsigned i = blockIdx.x * 256u + threadIdx.x;  // (T * K < 2^25)
  if (i >= (unsigned)a.T * (unsigned)a.K) return;
  const int r = a.dst_row[i], fk = a.first_k[i];
  if (r < 0) return;
  if (r >= a.rows || fk < 0 || fk >= a.K) {
    dev_set_error(a.error, EP_EBOUNDS);
    return;
  }
  a.index[r] = a.dst_row_g[i - i % (unsigned)a.K + fk];
}

int launch_gather_index(const GatherIndexArgs &a, void *stream) {
  const long long n = (long long)a.T * a.K;
  if (n <= 0) return 0;
  hipLaunchKernelGGL(gather_index_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

// The chain over the rows that the lanes in `ks` hold, ascending, for a top-k without an instance of its own: four loads
// in flight (4096 tokens x 4096 top-9 90 us, one load at a time 92; 2048 x 4096 top-16 72 and 76.  The plain combine,
// with a wave per slice and nothing else to do, is 3% faster without).
EP_DEV void fma_rows(float (&acc)[8], unsigned long long ks, int row, float wt, const u32x4 *y, int nvec, int v) {
  while (ks) {
    u32x4 ld[4];
    float w[4];
    int n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (!ks) break;
      const int k = __builtin_ctzll(ks);
      ks &= ks - 1;
      ld[j] = __builtin_nontemporal_load(y + (size_t)__builtin_amdgcn_readlane(row, k) * nvec + v);
      w[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), k));
      n = j + 1;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < n) fma8(acc, w[j], ld[j]);
  }
}

// First level of the hierarchical reduce: like the combine, but the K gathered
// rows of a token are summed per group and every group's sum is written to the
// group's own row.  Rows, weights and group leaders are wave-uniform.
// The sums are stored write-through, like the rows of a dispatch.  Deduplicated steps with y as it was / written just before, as
// the experts do (the copy's own time included), us: 4096 tokens x 7168 top-8 over 16 groups 327.5 and 500 (streaming stores 331.5
// and 519, plain 334.5 and 505), 8192 x 4096 376 and 576 (386 and 594, 384 and 580), 1024 x 7168 96.3 and 138.0 (100 and 141.8,
// 97.1 and 137.7).
template <int KT>
__global__ __launch_bounds__(256) void combine_partial_kernel(CombinePartialArgs a) {
  const int lane = lane_id();
  const unsigned item = blockIdx.x * (unsigned)a.group_waves + wave_id();
  const int t = (int)(item / (unsigned)a.parts), part = (int)(item % (unsigned)a.parts);
  if (t >= a.T) return;
  const int K = KT > 0 ? KT : a.K;
  int row = -1, fk = -1, prow = -1;
  float wt = 0.0f;
  if (lane < K) {
    row = a.dst_row[(size_t)t * K + lane];
    wt = a.w[(size_t)t * K + lane];
    fk = a.first_k[(size_t)t * K + lane];
    prow = a.dst_row_g[(size_t)t * K + lane];
    if (row < -1 || row >= a.y_rows || fk < -1 || fk >= K || (row >= 0 && fk < 0)) {
      dev_set_error(a.error, EP_EBOUNDS);
      row = -1;
    }
    if (row >= 0 && fk == lane && (prow < 0 || prow >= a.rows_g)) {
      dev_set_error(a.error, EP_EBOUNDS);
      row = -1;  // a leader without a valid row drops out; its followers find no open group below
    }
  }
  const unsigned long long vmask = __ballot(row >= 0);
  const unsigned long long leaders = __ballot(row >= 0 && fk == lane);
  if (vmask == 0) return;
  const int nvec = a.H >> 3;
  const int vi = part * 64 + lane;
  const u32x4 *y = (const u32x4 *)a.y;
  if constexpr (KT > 0) {
    if (vi >= nvec) return;
    int rows[KT], fks[KT];
    float ws[KT];
    u32x4 ld[KT];
    const int safe = __builtin_amdgcn_readlane(row, __builtin_ctzll(vmask));
#pragma unroll
    for (int k = 0; k < KT; ++k) {
      rows[k] = __builtin_amdgcn_readlane(row, k);
      fks[k] = __builtin_amdgcn_readlane(fk, k);
      ws[k] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wt), k));
      ld[k] = __builtin_nontemporal_load(y + (size_t)(rows[k] >= 0 ? rows[k] : safe) * nvec + vi);
    }
    // every group's chain first, the packed sums kept in registers; then the stores, together
    u32x4 res[KT];
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      if (!((leaders >> j) & 1)) continue;
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KT; ++k)
        if (rows[k] >= 0 && fks[k] == j) fma8(acc, ws[k], ld[k]);
      res[j] = u32x4{pack_bf16_rne(acc[0], acc[1]), pack_bf16_rne(acc[2], acc[3]), pack_bf16_rne(acc[4], acc[5]),
                     pack_bf16_rne(acc[6], acc[7])};
    }
#pragma unroll
    for (int j = 0; j < KT; ++j) {
      if (!((leaders >> j) & 1)) continue;
      const int pr = __builtin_amdgcn_readlane(prow, j);
      store_payload((u32x4 *)a.partial + (size_t)pr * nvec + vi, res[j]);
    }
  } else {
    unsigned long long lm = leaders;
    while (lm) {
      const int j = __builtin_ctzll(lm);
      lm &= lm - 1;
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      // (lanes past the row's end stay to the end: every lane's entry counts in the ballot)
      fma_rows(acc, __ballot(row >= 0 && fk == j), row, wt, y, nvec, min(vi, nvec - 1));
      const int pr = __builtin_amdgcn_readlane(prow, j);
      u32x4 o = {pack_bf16_rne(acc[0], acc[1]), pack_bf16_rne(acc[2], acc[3]),
                 pack_bf16_rne(acc[4], acc[5]), pack_bf16_rne(acc[6], acc[7])};
      if (vi < nvec) store_payload((u32x4 *)a.partial + (size_t)pr * nvec + vi, o);
    }
  }
}

// Waves per compute unit as in the combine, whose rule of 96 KB is 128 here, where every entry loads a row; top-4 and less have no
// limit, and four waves per workgroup.  The reduce alone, 12 / 14 / 16 / 20 waves, and four per workgroup with no limit, us:
//   top-8  4096 tokens x 7168 over 16 groups 153.1 / 156.1 / 155.8 / 157.7, 159.1, a tenth masked 138.3 / 140.2 / 140.7
//          / 142.3, 143.7, three tenths 107.3 / 101.5 / 100.4 / 100.5, 100.1, half 88.3 / 78.8 / 76.5 / 75.7, 76.3; 3000 x 7168
//          100.9 / 99.4 / 98.6 / 97.3, 98.3; over 8 groups 88.1 / 86.1 / 85.9 / 86.5, 86.9, a tenth masked 85.9 / 81.6 / 81.4 /
//          81.5, 81.9
//   top-7  13 / 14 / 16 / 20 waves 4096 x 7168 136.1 / 135.6 / 137.1 / 137.2, 140.6, half masked 75.4 / 75.4 / 72.0 /
//          67.8, 67.0
//   top-6  16 / 20 waves 4096 x 7168 114.6 / 116.1, 116.6; over 8 groups 93.9 / 93.2, 91.4; 8000 x 4096 129.7 / 130.8,
//          135.9
//   top-4  one per workgroup with 24 waves, and four with no limit 8000 x 4096 over 16 groups 75.8, 74.4, 1500 x 7168
//          27.9, 28.0
// (Loads for the entries that have a row only, as in the combine: 3000 x 7168 top-8 with 12 waves 118, with 20 102.)
constexpr int kPartialKb = 128;
int launch_combine_partial(const CombinePartialArgs &a0, void *stream) {
  if (a0.T <= 0) return 0;
  CombinePartialArgs a = a0;
  const int nvec = a.H / 8;
  a.parts = (nvec + 63) / 64;
  const long long items = (long long)a.T * a.parts;
  const int waves = a.K <= 4 ? 32 : a.K > 8 ? 24 : kPartialKb / a.K;  // (fma_rows has four loads in flight)
  const size_t lds = items >= 5ll * 256 * waves ? lds_for_waves(waves) : 0;
  a.group_waves = reduce_group_waves(items, a.K <= 4);
  const unsigned grid = (unsigned)((items + a.group_waves - 1) / a.group_waves);
  const dim3 block(64 * a.group_waves);
  hipStream_t st = (hipStream_t)stream;
  switch (a.K) {
    case 1: hipLaunchKernelGGL(combine_partial_kernel<1>, dim3(grid), block, lds, st, a); break;
    case 2: hipLaunchKernelGGL(combine_partial_kernel<2>, dim3(grid), block, lds, st, a); break;
    case 3: hipLaunchKernelGGL(combine_partial_kernel<3>, dim3(grid), block, lds, st, a); break;
    case 4: hipLaunchKernelGGL(combine_partial_kernel<4>, dim3(grid), block, lds, st, a); break;
    case 5: hipLaunchKernelGGL(combine_partial_kernel<5>, dim3(grid), block, lds, st, a); break;
    case 6: hipLaunchKernelGGL(combine_partial_kernel<6>, dim3(grid), block, lds, st, a); break;
    case 7: hipLaunchKernelGGL(combine_partial_kernel<7>, dim3(grid), block, lds, st, a); break;
    case 8: hipLaunchKernelGGL(combine_partial_kernel<8>, dim3(grid), block, lds, st, a); break;
    default: hipLaunchKernelGGL(combine_partial_kernel<0>, dim3(grid), block, lds, st, a); break;
  }
  return (int)hipGetLastError();
}

}  // namespace ep
