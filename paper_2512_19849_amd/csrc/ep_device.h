// Device-side helpers shared by the HIP kernels of libep.so (gfx950): the GPU end of the GPU->CPU FIFO
// channels (Push, Check-completion, Drain), the payload store and its completion wait, the FP8
// quantiser, and small wave-level utilities.  Everything here is inlined into the kernels.
#ifndef EP_DEVICE_H_
#define EP_DEVICE_H_
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "ep_internal.h"

namespace ep {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

#define EP_DEV __device__ __forceinline__

// ---------------------------------------------------------------- utilities
EP_DEV void dev_set_error(int *err, int code) {
  // Sticky error word in pinned host memory; any failing lane may write it.
  __hip_atomic_store(err, code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

EP_DEV int lane_id() { return threadIdx.x & 63; }

// This wave's place in its workgroup, in a scalar register: what is worked out from it (token, part of the row, addresses)
// is then scalar work too.  As a vector value, the 64-bit division of a wave's number alone was 150 vector instructions ahead
// of the combine's first load.  Whole steps do not show it beyond what two runs differ by (vector / scalar, us: 128 tokens x
// 7168 over 32 sources 34.2 / 34.8, 8192 x 4096 with a command per row 253.3 / 253.5, deduplicated 4096 x 7168 355.8 / 355.4).
EP_DEV unsigned wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// ------------------------------------------------- FIFO channel, GPU side
// Push (Section 3.1, "Channel APIs"): reserve the next Idx of the channel with
// one device-scope atomic on the tail (which lives in device memory), wait for
// room using the device-resident cached copy of the head and re-reading the
// host copy over PCIe only when that cache says "full", then publish the
// 16-byte command with a single store.  Returns Idx, or ~0 after a timeout.
EP_DEV unsigned long long ring_publish(const RingDev &r, unsigned c, unsigned long long idx, unsigned w0, unsigned w1,
                                       unsigned w2, unsigned w3);
EP_DEV unsigned long long ring_push(const RingDev &r, unsigned c, unsigned w0, unsigned w1,
                                    unsigned w2, unsigned w3) {
  const unsigned long long idx =
      __hip_atomic_fetch_add(&r.tail[c], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return ring_publish(r, c, idx, w0, w1, w2, w3);
}

// Push for a whole wave whose lanes hold one command each (or none: `active`), called by all 64 lanes together.  Lanes that
// aim at the same channel share ONE atomic on its tail - the first of them reserves a run of Idx for all, the others take
// their place in the run (atomics on one address serialise in the L2, and a per-token dispatch sends tens of thousands of
// commands through a handful of tails).  Then the commands change lanes through LDS (`scratch`, kSortScratch) so that lane
// order is (channel, Idx) order: neighbouring lanes store neighbouring slots, and the memory pipeline turns the slots of one
// 64-byte line into one write.  A line of host memory that the proxy is polling costs the PCIe root a round of coherence
// traffic per write that lands in it, whatever the size of the write.
// (The check for room reads the cached head after the reservation: read together with it, it is older, calls the channel
// full more often, and a prefill dispatch of 65536 commands took 178 us instead of 162.)
// In two halves, so that a caller can have other round trips under way with the second.
constexpr unsigned kSortScratch = 2048;  // bytes
struct SortedRun {
  unsigned long long idx;  // this lane's Idx
  int place, n;            // its place among the n commands of the wave
};
EP_DEV SortedRun ring_reserve_sorted(const RingDev &r, bool active, unsigned c) {
  const int me = lane_id();
  const unsigned long long act = __ballot(active);
  SortedRun run{0ull, 0, (int)__popcll(act)};
  if (act == 0ull) return run;
  unsigned long long same = 0ull;
  int less = 0;
  for (unsigned long long m = act; m;) {  // once per distinct channel
    const unsigned cj = (unsigned)__builtin_amdgcn_readlane((int)c, __builtin_ctzll(m));
    const unsigned long long mj = __ballot(active && c == cj);
    if (cj == c) same = mj;
    if (cj < c) less += __popcll(mj);
    m &= ~mj;
  }
  const int leader = (active && same) ? __builtin_ctzll(same) : 0;
  const int before = __popcll(same & ((1ull << me) - 1ull));
  unsigned long long base = 0ull;
  if (active && me == leader)
    base = __hip_atomic_fetch_add(&r.tail[c], (unsigned long long)__popcll(same), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  base = ((unsigned long long)(unsigned)__shfl((int)(base >> 32), leader) << 32) | (unsigned)__shfl((int)base, leader);
  run.idx = base + (unsigned long long)before;
  run.place = less + before;
  return run;
}
EP_DEV void ring_publish_sorted(const RingDev &r, bool active, const SortedRun &run, unsigned c, unsigned w0, unsigned w1,
                                unsigned w2, unsigned w3, u32x4 *scratch) {
  if (run.n == 0) return;
  const int me = lane_id();
  if (active) {
    scratch[run.place] = u32x4{w0, w1, w2, w3};
    scratch[64 + run.place] = u32x4{c, (unsigned)run.idx, (unsigned)(run.idx >> 32), 0u};
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (me < run.n) {
    const u32x4 w = scratch[me], q = scratch[64 + me];
    ring_publish(r, q.x, ((unsigned long long)q.z << 32) | q.y, w.x, w.y, w.z, w.w);
  }
  __builtin_amdgcn_wave_barrier();  // (the next round writes the scratch again)
}
EP_DEV void ring_push_sorted(const RingDev &r, bool active, unsigned c, unsigned w0, unsigned w1, unsigned w2,
                             unsigned w3, u32x4 *scratch) {
  ring_publish_sorted(r, active, ring_reserve_sorted(r, active, c), c, w0, w1, w2, w3, scratch);
}

// Second half of a Push: wait for room for the reserved Idx, then publish the command - or N of them, with Idx in a row.
// `head` is a head of the channel read before, or what ring_head returns.
EP_DEV unsigned long long ring_head(const RingDev &r, unsigned c) {
  return __hip_atomic_load(&r.cached_head[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One 16-byte store straight to host memory (system scope); not waited for here, see store_payload.
EP_DEV void ring_store(const RingDev &r, unsigned c, unsigned long long idx, u32x4 v) {
  const unsigned gen = (((unsigned)(idx >> r.log2_entries)) & 1u) ^ 1u;
  v[0] |= gen << 31;
  v[3] |= gen << 31;
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" ::"v"((u32x4 *)r.slots + (size_t)c * r.entries +
                                                              (size_t)(idx & (r.entries - 1))),
               "v"(v)
               : "memory");
}
template <int N>
EP_DEV unsigned long long ring_publish_run(const RingDev &r, unsigned c, unsigned long long idx, unsigned long long head,
                                           const u32x4 &first, const u32x4 &second) {
  unsigned long long result = idx, t0 = 0;
  int next = 0;
  bool stalled = false;
  // Lanes of one wavefront push side by side, and the proxy consumes a channel in Idx order: a lane
  // whose Idx already fits must publish its command without waiting for a neighbour whose Idx does
  // not fit yet (that neighbour may be waiting for the very slot this lane has to fill).  So the
  // store sits INSIDE the wave-wide loop, and the loop ends when every active lane is done.
  do {
    if (next < N) {
      if (idx + next - head < r.entries) {
        ring_store(r, c, idx + next, next == 0 ? first : second);
        ++next;
        stalled = false;  // (the next command's wait is its own: a limit and a count for each)
      } else {
        // Full: wait for the proxy to pop.  Thousands of lanes can be waiting on one channel, and
        // each re-read of the head is a PCIe round trip, so only the lane that holds the channel's
        // refresh lock goes to host memory; everyone else watches the device-side copy it updates.
        if (!stalled) {
          stalled = true;
          t0 = wall_clock64();
          __hip_atomic_fetch_add(r.stalls, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (__hip_atomic_exchange(&r.refresh_lock[c], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
          const unsigned long long h =
              __hip_atomic_load(&r.head[c * kHeadStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          __hip_atomic_fetch_max(&r.cached_head[c], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&r.refresh_lock[c], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        head = ring_head(r, c);
        if (idx + next - head >= r.entries) {
          if (wall_clock64() - t0 > r.timeout_ticks) {
            dev_set_error(r.error, EP_ETIMEOUT);
            result = ~0ull;
            next = N;
          } else {
            __builtin_amdgcn_s_sleep(32);
          }
        }
      }
    }
  } while (__ballot(next < N) != 0ull);
  return result;
}
EP_DEV unsigned long long ring_publish(const RingDev &r, unsigned c, unsigned long long idx, unsigned w0, unsigned w1,
                                       unsigned w2, unsigned w3) {
  const u32x4 v = {w0, w1, w2, w3};
  return ring_publish_run<1>(r, c, idx, ring_head(r, c), v, v);
}

// For the lanes with `active`, which have published a command with Idx: the one with the first of half a ring reads the head for
// all, so that the device-side copy keeps up with the proxy.  Left until the copy calls the ring full, as it does once per trip
// round the ring whether the proxy is behind or not, the read over PCIe is one that everybody with a command for the channel
// waits for.  To be called when nothing else of the wave is waited for, and not towards the end of a kernel, which the read (10
// us and more behind a chip full of stores) would prolong.  Every half ring is as good as every quarter, an eighth costs 1%.
EP_DEV void ring_refresh_ahead(const RingDev &r, bool active, unsigned c, unsigned long long idx) {
  if (!active || ((unsigned)idx & ((r.entries >> 1) - 1u)) != 0u) return;
  const unsigned long long h = __hip_atomic_load(&r.head[c * kHeadStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __hip_atomic_fetch_max(&r.cached_head[c], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

EP_DEV unsigned long long readlane64(unsigned long long v, int lane) {
  return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(v >> 32), lane) << 32) |
         (unsigned)__builtin_amdgcn_readlane((int)v, lane);
}

// Push for a whole wave some lanes of which (`active`) hold two commands for one channel, a Write and the Atomic behind it.
// One reservation for both, the heads read together with it; then the wave stores a lane's pair at a time, from two lanes, so
// that it arrives at the host as one write (see ring_push_sorted).  What finds its channel full publishes lane by lane.
// The proxy misses its caches once per write, and takes a quarter of a microsecond for it.  Whole steps, one Push after the
// other / pairs, us: sequenced chunks of 1531 tokens x 5120 top-6 64 / 58 (both stores of a pair from one lane 61), 2048 x
// 2048 top-4 48 / 43; ring-buffer channels 4096 x 7168 442 / 427, 4096 x 4096 in FP8 244 / 218, 600 x 2048 131 / 112.
EP_DEV void ring_push_pairs(const RingDev &r, bool active, unsigned c, const u32x4 &write, const u32x4 &atomic) {
  const unsigned long long act = __ballot(active);
  if (act == 0ull) return;
  unsigned long long idx = 0ull, head = 0ull;
  if (active) {
    idx = __hip_atomic_fetch_add(&r.tail[c], 2ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    head = ring_head(r, c);
  }
  if (__ballot(active && idx + 1ull - head >= r.entries) != 0ull) {
    if (active) ring_publish_run<2>(r, c, idx, head, write, atomic);
    return;
  }
  const int me = lane_id();
  for (unsigned long long m = act; m; m &= m - 1) {
    const int k = __builtin_ctzll(m);
    const unsigned ck = (unsigned)__builtin_amdgcn_readlane((int)c, k);
    const unsigned long long ik = readlane64(idx, k);
    u32x4 v;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int w = __builtin_amdgcn_readlane((int)write[j], k), x = __builtin_amdgcn_readlane((int)atomic[j], k);
      v[j] = (unsigned)(me == 0 ? w : x);
    }
    if (me < 2) ring_store(r, ck, ik + (unsigned)me, v);
  }
}

// Check-completion(Idx): has the proxy popped command idx of channel c?
// Blocks (bounded) until it has; used after a Drain.
EP_DEV void wait_for_own_stores();
EP_DEV bool ring_wait_completion(const RingDev &r, unsigned c, unsigned long long idx) {
  // the command has to have left before it can be popped: a poll issued together with the Push store
  // only finds the old head, and the next poll comes a sleep and a PCIe round trip later
  wait_for_own_stores();
  const unsigned long long t0 = wall_clock64();
  for (;;) {
    unsigned long long head =
        __hip_atomic_load(&r.head[c * kHeadStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (head > idx) return true;
    if (wall_clock64() - t0 > r.timeout_ticks) {
      dev_set_error(r.error, EP_ETIMEOUT);
      return false;
    }
    __builtin_amdgcn_s_sleep(32);
  }
}

// Payload rows are stored write-through at system scope (sc0 sc1): when such a store is
// acknowledged the bytes are in memory, visible to every XCD's L2 and to a PCIe reader, which is
// what a transfer command promises about the rows it names.  A wave therefore only has to wait
// for its own stores (vmcnt) before it touches a counter or pushes a command; no L2 write-back
// is needed, and the counters can be relaxed device-scope atomics.  Measured on MI355X the
// write-through stores stream as fast as non-temporal ones, whereas a device-scope release fence
// per wave (L2 write-back) made the dispatch 4-8x slower.
// The store is written out as the instruction itself: the way to get these cache bits from C++ is
// a volatile access, and the compiler follows EVERY volatile store with a wait for all outstanding
// memory operations - a wave would then hand the memory system one kilobyte at a time (dispatch
// 91 -> 87 us without those waits).  The compiler does not count these stores, so the wait that
// orders them is explicit as well.
EP_DEV void store_payload(u32x4 *p, const u32x4 &v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc0 sc1" ::"v"(p), "v"(v) : "memory");
}

// All stores of this wave are acknowledged after this (hardware wait, then a compiler barrier).
EP_DEV void wait_for_own_stores() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt and lgkmcnt left alone
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
}

// Kernel epilogue with EP_CMD_DRAIN: the last workgroup of the grid to finish pushes a Drain on
// every channel and blocks on Check-completion for each (Section 3.1: Drain and Barrier are blocking
// on the GPU side).  Every wave of every workgroup must call this.
// "Last to finish" is counted per workgroup and in two levels (groups of kDrainGroup workgroups,
// then groups): atomics on ONE address serialise in the L2 at about 8 ns each, and one count per
// wave of a 32768-wave grid added 270 us to the kernel.  done_cnt: [1 + groups] scratch, zero
// between launches (the counters reset themselves).
constexpr unsigned kDrainGroup = 64;
EP_DEV void drain_all_channels(const RingDev &ring, unsigned *done_cnt, unsigned src, int lane) {
  wait_for_own_stores();  // this wave's commands are in their rings ...
  __syncthreads();        // ... and so are those of every wave of the workgroup
  if (threadIdx.x >= 64) return;
  unsigned last = 0;
  if (lane == 0) {
    const unsigned block = blockIdx.y * gridDim.x + blockIdx.x, blocks = gridDim.x * gridDim.y;
    const unsigned group = block / kDrainGroup, ngroups = (blocks + kDrainGroup - 1) / kDrainGroup;
    const unsigned gsize = min(kDrainGroup, blocks - group * kDrainGroup);
    if (__hip_atomic_fetch_add(&done_cnt[1 + group], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gsize) {
      __hip_atomic_store(&done_cnt[1 + group], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__hip_atomic_fetch_add(&done_cnt[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == ngroups) {
        __hip_atomic_store(&done_cnt[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = 1;
      }
    }
  }
  if (!__builtin_amdgcn_readfirstlane(last)) return;
  for (unsigned c = lane; c < ring.channels; c += 64) {
    const unsigned long long idx = ring_push(ring, c, cmd_w0(EP_OP_DRAIN, src, 0, 0), 0u, 0u, 0u);
    if (idx != ~0ull) ring_wait_completion(ring, c, idx);
  }
}

// ---------------------------------------------------------- wave utilities
EP_DEV int wave_inclusive_scan(int v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(v, d);
    if (lane >= d) v += u;
  }
  return v;
}

// Sum over the 64 lanes, in every lane: adds within rows of 16 lanes, then across the four rows (DPP moves: no LDS).
EP_DEV int wave_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true);  // row_half_mirror
  v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true);  // row_mirror
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}

// One launch, with the kernel's own begin / end timestamps delivered into the caller's events when asked for.
template <class Kernel, class Args>
static inline void launch_kernel(Kernel kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, void *ev_start,
                                 void *ev_stop, const Args &a) {
  if (ev_start || ev_stop)
    hipExtLaunchKernelGGL(kernel, grid, block, (unsigned)lds, st, (hipEvent_t)ev_start, (hipEvent_t)ev_stop, 0, a);
  else
    hipLaunchKernelGGL(kernel, grid, block, lds, st, a);
}

// ------------------------------------------------------------ FP8 quantiser
EP_DEV float bf16_lo(unsigned d) { return __uint_as_float(d << 16); }
EP_DEV float bf16_hi(unsigned d) { return __uint_as_float(d & 0xFFFF0000u); }

// Two floats -> two E4M3 codes (round to nearest even, saturate to +-448)
// in the low or high half of a dword.  The clamp is exact, so the hardware
// conversion never sees a value beyond the largest finite code.
template <bool HI>
EP_DEV unsigned cvt2_e4m3(float x, float y, unsigned old) {
  x = __builtin_amdgcn_fmed3f(x, 448.0f, -448.0f);
  y = __builtin_amdgcn_fmed3f(y, 448.0f, -448.0f);
  return (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(x, y, (int)old, HI);
}

// A lane owns 16 consecutive channels (two 16-byte loads, one 16-byte store of
// codes); 8 adjacent lanes own one 128-channel block and share its amax through
// three xor-shuffles.  scale = amax/448 and inv = 448/amax are IEEE divisions.
// Every lane of the wave must call this (lanes past the row's end with zeros).
EP_DEV void quant16(const u32x4 &lo, const u32x4 &hi, u32x4 &q, float &scale_out) {
  float f[16];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f[2 * j] = bf16_lo(lo[j]);
    f[2 * j + 1] = bf16_hi(lo[j]);
    f[8 + 2 * j] = bf16_lo(hi[j]);
    f[8 + 2 * j + 1] = bf16_hi(hi[j]);
  }
  float amax = 0.0f;
#pragma unroll
  for (int j = 0; j < 16; ++j) amax = fmaxf(amax, fabsf(f[j]));
  amax = fmaxf(amax, __shfl_xor(amax, 1));
  amax = fmaxf(amax, __shfl_xor(amax, 2));
  amax = fmaxf(amax, __shfl_xor(amax, 4));
  float scale = 1.0f, inv = 1.0f;
  if (amax >= 0x1p-100f) {
    scale = amax / 448.0f;
    inv = 448.0f / amax;
  }
  scale_out = scale;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    unsigned d = cvt2_e4m3<false>(f[4 * j] * inv, f[4 * j + 1] * inv, 0u);
    q[j] = cvt2_e4m3<true>(f[4 * j + 2] * inv, f[4 * j + 3] * inv, d);
  }
}

}  // namespace ep
#endif  // EP_DEVICE_H_
