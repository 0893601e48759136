// Ring-buffer communication channels of the high-throughput mode: one or several workgroups per token slice play the
// sending and the receiving end in turns, chunk slots reused under head/tail flow control.
#include <cstddef>
#include <type_traits>

#include "ep_device.h"

namespace ep {

// ------------------------------------------- ring-buffer channels (HT mode)
// Section 3.3 ("partial ordering"): tokens travel through rings of chunk slots; the sender may reuse
// a slot only after the receiver released it (head), the receiver may read it only after it was
// announced (tail); Write, tail Atomic and head Atomic are sequenced per channel and pass through the
// proxy.
// A workgroup owns the channels of a token slice, or some of them (see launch_ht_ring), and plays
// both ends of them in turns: a sending step (every wavefront takes a token, keeps its row in
// registers and stores it into the slot of each of its destinations that is known to be free, then
// announces the chunks it completed) and a receiving step (a sweep over the tails, the announced
// rows move to their final place, the slots are released).  Neither step waits for the other end: a
// wavefront whose slot is still occupied keeps its claimed position and tries again after the next
// sweep.  A workgroup therefore depends on nothing but the proxy, whatever the grid size and
// however many workgroups are resident, and every compute unit has rows to store all the time.
// On this hardware one counter tracks a wave's outstanding loads AND stores, so waiting for any load
// also waits for every store issued before it; the sending step is shaped around that: all of a
// token's metadata in one load, the row in one batch of loads, then nothing but stores.
// Every wait is bounded; without progress for the time limit the workgroup gives up with an error.
constexpr int kHtMaxRanks = 256, kHtMaxSlots = 4096, kHtHeader = 128;

struct HtShared {
  int total[kHtMaxRanks];      // rows of channel (slice, r) in this dispatch
  // sending end
  int fill[kHtMaxRanks];       // positions handed out
  unsigned seen[kHtMaxRanks];  // rows known to be released in this dispatch (cached head)
  int lock[kHtMaxRanks];       // who refreshes seen[r] over PCIe
  unsigned seqf[kHtMaxRanks];  // the channel's forward sequence number before this dispatch
  unsigned cumf[kHtMaxRanks];  // rows the channel carried before this dispatch (sender's count)
  int done[kHtMaxSlots];       // rows stored per (r, slot)
  // receiving end
  int next[kHtMaxRanks];       // next chunk to consume
  int lo[kHtMaxRanks], hi[kHtMaxRanks];  // chunks [lo, hi) are consumed in the current sweep
  unsigned seqr[kHtMaxRanks];  // the channel's reverse sequence number before this dispatch
  unsigned cumr[kHtMaxRanks];  // rows the channel carried before this dispatch (receiver's count)
  bool mine[kHtMaxRanks];  // the channel of slice and rank is this workgroup's (see ht_share)
  int abort, remaining, progress, idle, announced, split;
};

#define HT_LD(p) __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
#define HT_ST(p, v) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)

EP_DEV bool ht_valid(const HtRingArgs &a, int e, int row) {
  return e >= 0 && e / a.E_loc < a.R && row >= 0 && row < a.recv_rows;
}

// Which of the slice's channels are workgroup `part`'s: ranks in descending order of their rows are dealt out to the `split`
// workgroups there and back (0 1 1 0 0 1 ...), so that each moves about the same number.  All of them count the same table and
// arrive at the same shares; a channel's state is read and written back by whoever has it in this dispatch.  Called by every
// thread, with the rows of all ranks in sh.total; clears those of the others.
// A dispatch ends with its slowest workgroup.  By rank number (r mod split) a skewed routing gave one half of the workgroups 165
// rows and the other 91 (4096 tokens x 7168 top-8, 128 slices; now 128 and 128, the kernel 313 us, now 297).  Whole steps, by
// rank number / by rows, us: this one 405 / 400, 2048 tokens 215 / 209, 3000 x 5120 over 64 slices 241 / 231, uniform routing
// 394 / 391.
EP_DEV void ht_share(const HtRingArgs &a, HtShared &sh, int split, int part) {
  for (int r = threadIdx.x; r < a.R; r += blockDim.x) {
    int ahead = 0;  // ranks in front of r in descending order
    for (int j = 0; j < (split > 1 ? a.R : 0); ++j) ahead += sh.total[j] > sh.total[r] || (sh.total[j] == sh.total[r] && j < r);
    const int at = ahead % split;
    sh.mine[r] = ((ahead / split) & 1 ? split - 1 - at : at) == part;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < a.R; r += blockDim.x)
    if (!sh.mine[r]) sh.total[r] = 0;
}

// B 16-byte vectors per lane of a row, starting at vector v0: loads in flight together, stores
// back to back.  The slots are stored write-through, the received rows plainly.  With the streaming hint on both, steps of
// 235 MB of rows and more took 2 to 6% less (4096 tokens x 7168 top-8, 128 slices: 474 us, without 489), steps of up to
// 110 MB 6 to 12% more (1024 x 4096, 64 slices: 155, without 139), and with a read of the received rows behind it a step of
// 470 MB over 256 slices 3% more (555, without 537).
template <bool STREAM, int B>
EP_DEV void ht_load_piece(u32x4 (&r)[B], const u32x4 *src, int v0, int nvec) {
#pragma unroll
  for (int i = 0; i < B; ++i)
    if (v0 + i * 64 < nvec) r[i] = STREAM ? __builtin_nontemporal_load(src + v0 + i * 64) : src[v0 + i * 64];
}
template <bool THROUGH, int B>
EP_DEV void ht_store_piece(const u32x4 (&r)[B], u32x4 *dst, int v0, int nvec) {
#pragma unroll
  for (int i = 0; i < B; ++i)
    if (v0 + i * 64 < nvec) {
      if (THROUGH) store_payload(dst + v0 + i * 64, r[i]);
      else dst[v0 + i * 64] = r[i];
    }
}

// The channels' state, read from the kernel's arguments where it is needed: kept in scalar registers from the kernel's start
// on, it makes them spill.
EP_DEV RingDev ht_fifo() {
  auto p = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  RingDev r;
  __builtin_memcpy(&r, (const char *)p + offsetof(HtRingArgs, fifo), sizeof(r));
  return r;
}

// What a wave remembers of the token it is sending: lane k owns the token's k-th entry.
struct HtToken {
  unsigned long long pend;  // entries claimed but not stored yet (wave-uniform)
  int p;                    // lane k: the position claimed in its channel
};

// One token: claim a position per valid entry (unless the wave comes back to a token it could not
// finish), find the entries whose slot is free, load the row once and store it to each of them,
// write the headers, wait once for all the stores, count the rows and announce every chunk that
// became complete (Write, then the tail Atomic).  Returns true when the token is finished; false
// when some of its slots are still occupied (the wave has stored and counted what it could).
constexpr int kHtPiece = 16;  // vectors per lane held in registers (bf16 rows up to 8192 channels in one piece)
EP_DEV bool ht_send_token(const HtRingArgs &a, HtShared &sh, int c, int t, HtToken &tk) {
  const int lane = lane_id();
  int e = -1, row = -1;
  if (lane < a.K) {
    e = a.idx[(size_t)t * a.K + lane];
    row = a.dst_row[(size_t)t * a.K + lane];
  }
  const bool valid = lane < a.K && ht_valid(a, e, row) && sh.mine[e / a.E_loc];
  const int r = valid ? e / a.E_loc : 0, chan = c * a.R + r;
  if (tk.pend == 0ull) {  // a new token: positions are handed out in arrival order
    tk.p = valid ? __hip_atomic_fetch_add(&sh.fill[r], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0;
    tk.pend = __ballot(valid);
    if (tk.pend == 0ull) return true;
  }
  const bool mine = (tk.pend >> lane) & 1ull;
  const int chunk = tk.p >> 5;
  bool occupied = false;
  if (mine && chunk >= a.W) {
    const unsigned need = 32u * (unsigned)(chunk - a.W + 1);
    if (HT_LD(&sh.seen[r]) < need) {
      // one PCIe read on behalf of every wave of the workgroup that needs this channel's head
      if (__hip_atomic_exchange(&sh.lock[r], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 0) {
        const unsigned v =
            (unsigned)__hip_atomic_load(a.head + chan, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) - sh.cumf[r];
        __hip_atomic_fetch_max(&sh.seen[r], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        HT_ST(&sh.lock[r], 0);
      }
      occupied = HT_LD(&sh.seen[r]) < need;
    }
  }
  const bool go = mine && !occupied;
  const unsigned long long ready = __ballot(go);
  if (ready == 0ull) return false;
  // byte offset of the entry's row in the ring (slot header included), split for readlane
  const unsigned long long off =
      ((unsigned long long)chan * a.W + chunk % a.W) * a.slot_bytes + kHtHeader + (unsigned long long)(tk.p & 31) * a.row_bytes;
  const unsigned off_lo = (unsigned)off, off_hi = (unsigned)(off >> 32);
  const u32x4 *xrow = (const u32x4 *)((const char *)a.x + (size_t)t * 2u * (unsigned)a.H);
  if (a.payload == EP_BF16) {
    const int nvec = a.H >> 3;
    for (int v0 = lane; v0 < nvec; v0 += 64 * kHtPiece) {
      u32x4 regs[kHtPiece];
      ht_load_piece<false, kHtPiece>(regs, xrow, v0, nvec);
      for (unsigned long long m = ready; m; m &= m - 1) {
        const int k = __builtin_ctzll(m);
        const unsigned long long o = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)off_hi, k) << 32) |
                                     (unsigned)__builtin_amdgcn_readlane((int)off_lo, k);
        ht_store_piece<true, kHtPiece>(regs, (u32x4 *)((char *)a.ring_buf + o), v0, nvec);
      }
    }
  } else {
    // FP8 message: the row's E4M3 codes, then one fp32 scale per 128 channels (Section 2.1: the ~7 KB token); quantised once
    // per token, stored to every destination.  Rows of up to 8192 channels are quantised whole before the first store, two
    // groups of channels per lane at a time (more, and the registers do not last), and their scales leave as one store: a
    // second half would wait for the stores of the first.  Whole steps, four groups and then the next four, scales 32 bytes at
    // a time, and in the receiving step behind the codes / this, us: 4096 tokens x 7168 top-8, 128 slices 299 / 293, 2048
    // tokens 204 / 194, 3000 x 8064 over 256 264 / 246, 4096 x 4096 212 / 202, 1024 x 3072 over 64 91 / 89. Groups that a
    // narrow row does not have are passed over: with all eight quantised whatever the width 4096 x 1024 over 64 slices takes
    // 207, with four 196, like this 178; 2000 x 2048 117, 121 and 110; 4096 x 7168 the same.
    constexpr int kPairs = 8;  // (64 blocks: a lane's scale each)
    const int npair = a.H >> 4;
    for (int p0 = 0; p0 < npair; p0 += 64 * kPairs) {
      u32x4 q[kPairs];
      float sc[kPairs];
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        if (i && i % 2 == 0)  // (holds the next loads back)
          asm volatile("" : "+v"(q[i - 1]), "+v"(q[i - 2]), "+v"(sc[i - 1]), "+v"(sc[i - 2])::"memory");
        const int first = __builtin_amdgcn_readfirstlane(p0 + i * 64);
        q[i] = u32x4{0, 0, 0, 0};
        sc[i] = 0.0f;
        if (first >= npair) continue;  // (a narrow row has nothing left to quantise)
        u32x4 lo = {0, 0, 0, 0}, hi = {0, 0, 0, 0};
        if (first + lane < npair) {
          const char *at = (const char *)xrow + (size_t)first * 32u;
          lo = *(const u32x4 *)(at + lane * 32u);
          hi = *(const u32x4 *)(at + lane * 32u + 16u);
        }
        quant16(lo, hi, q[i], sc[i]);
      }
      float scale = 0.0f;  // lane b: block b of these
#pragma unroll
      for (int i = 0; i < kPairs; ++i) {
        const float u = __shfl(sc[i], (lane & 7) * 8);
        if (lane >> 3 == i) scale = u;
      }
      for (unsigned long long m = ready; m; m &= m - 1) {
        const int k = __builtin_ctzll(m);
        const unsigned long long o = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)off_hi, k) << 32) |
                                     (unsigned)__builtin_amdgcn_readlane((int)off_lo, k);
        char *dst = (char *)a.ring_buf + o;
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
          const int p = p0 + i * 64 + lane;
          if (p < npair) store_payload((u32x4 *)dst + p, q[i]);
        }
        const int b = (p0 >> 3) + lane;
        if (b < a.H >> 7)
          __hip_atomic_store((float *)(dst + a.H) + b, scale, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
  const int n = tk.p >> 5, slot_row = tk.p & 31, w = n % a.W;
  if (go) {
    int *hdr = (int *)((char *)a.ring_buf + ((unsigned long long)chan * a.W + w) * a.slot_bytes);
    __hip_atomic_store(hdr + slot_row, row, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  wait_for_own_stores();
  int sz = 0;
  bool whole = false;  // this lane's row was the last one of its chunk
  if (go) {
    sz = min(kChunkRows, sh.total[r] - (n << 5));
    whole = __hip_atomic_fetch_add(&sh.done[r * a.W + w], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + 1 == sz;
    if (whole) HT_ST(&sh.done[r * a.W + w], 0);
  }
  if (__ballot(whole) != 0ull) {
    const unsigned seq = sh.seqf[r] + 2u * (unsigned)n, len = (unsigned)kHtHeader + (unsigned)sz * a.row_bytes;
    const unsigned w0 = cmd_w0(EP_OP_RING, a.src, (unsigned)r, (unsigned)c);
    const RingDev fifo = ht_fifo();
    ring_push_pairs(fifo, whole, (unsigned)chan % fifo.channels,
                    u32x4{w0, ((unsigned)EP_RING_WRITE << 30) | ((unsigned)(sz - 1) << 24) | (len >> 4), seq,
                          (unsigned)((((size_t)chan * a.W + w) * a.slot_bytes) >> 4)},
                    u32x4{w0, ((unsigned)EP_RING_TAIL << 30) | (unsigned)sz, seq + 1u, 0u});
  }
  if (lane == 0) HT_ST(&sh.progress, 1);
  tk.pend &= ~ready;
  return tk.pend == 0ull;
}

// One sending step of a wavefront: the slice's tokens are dealt to the waves round-robin; a step
// takes about kHtStepRows rows' worth of them (q counts the wave's finished tokens).  Returns true
// when the wave has nothing left to send.
constexpr int kHtStepRows = 16;
EP_DEV bool ht_send_step(const HtRingArgs &a, HtShared &sh, int c, int t0, int ntok, int &q, HtToken &tk) {
  const int wave = wave_id(), nwaves = blockDim.x >> 6;
  const int budget = max(1, kHtStepRows * sh.split / a.K);
  for (int j = 0; j < budget; ++j) {
    const int tt = wave + q * nwaves;
    if (tt >= ntok) return true;
    if (!ht_send_token(a, sh, c, t0 + tt, tk)) return false;
    ++q;
  }
  return false;
}

// One receiving step of the workgroup: a sweep over the slice's tails, the announced rows move to
// the rows their headers name, the consumed slots are released.  Called by every thread.
EP_DEV void ht_receive_step(const HtRingArgs &a, HtShared &sh, int c) {
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id(), nwaves = blockDim.x >> 6;
  const bool fp8 = a.payload != EP_BF16;
  const int nvec = fp8 ? a.H >> 4 : a.H >> 3;  // 16-byte vectors of payload per row
  const unsigned rb = a.row_bytes;
  // which chunks have been announced since the last sweep (at most W per channel)
  for (int r = tid; r < a.R; r += blockDim.x) {
    const int tot = sh.total[r], nch = (tot + 31) >> 5, n0 = sh.next[r];
    int hi = n0;
    if (n0 < nch) {
      const unsigned avail =
          (unsigned)__hip_atomic_load(a.tail + c * a.R + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) - sh.cumr[r];
      while (hi < nch && hi - n0 < a.W && avail >= (unsigned)min((hi + 1) << 5, tot)) ++hi;
    }
    sh.lo[r] = n0;
    sh.hi[r] = hi;
    if (hi > n0) sh.announced = 1;
  }
  __syncthreads();
  if (!sh.announced) return;
  // What a tail announces reached memory from outside this compute unit's view (a network adapter in the paper; here the sending
  // step's write-through stores), possibly into lines a cache still holds from the slot's previous use: drop those before the
  // first read of the sweep (the acquire that pairs with the tail).  It empties the XCD's L2, so one wave does it for all, and
  // none on idle sweeps.  A wave's own loads are served behind its invalidate; for the others' the barrier alone says nothing, as
  // the invalidate may still be on its way when its wave arrives there.  So that wave loads a word behind it, through the caches it
  // empties, and waits for the word: by then the invalidate is through this compute unit's L1 and ahead of every later load in
  // its queues to the L2.  Whole steps, by every wave / by one, us: 4096 tokens x 7168 top-8, 128 slices 423 / 403, 3000 x 5120,
  // 256 slices 270 / 239, 1024 x 4096, 64 slices 107 / 98, 600 x 2048 top-4 63.8 / 62.5; 2048 x 7168 in FP8, 128 slices 204 / 194.
  if (wave == 0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    const int behind = __hip_atomic_load(a.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(behind) : "memory");
  }
  __syncthreads();
  if (tid == 0) sh.announced = 0;
  // move their rows to where the header says; rows are dealt out to the waves round-robin
  int q = 0;
  for (int r = 0; r < a.R; ++r) {
    const int lo = sh.lo[r], hi = sh.hi[r];
    for (int n = lo; n < hi; ++n) {
      const int sz = min(kChunkRows, sh.total[r] - (n << 5));
      const char *slot = (const char *)a.ring_buf + ((size_t)(c * a.R + r) * a.W + n % a.W) * a.slot_bytes;
      // this wave's rows of the chunk: j = first, first + nwaves, ... (rows are dealt round-robin over all chunks)
      const int first = (wave - q % nwaves + nwaves) % nwaves;
      q += sz;
      if (first >= sz) continue;
      // one load brings the destination rows of the whole chunk; the rows are then moved two at a
      // time so that the loads of both are in flight together
      const int hdr = lane < sz ? __builtin_nontemporal_load((const int *)slot + lane) : -1;
      const size_t out_stride = fp8 ? (size_t)a.H : (size_t)rb;
      for (int j = first; j < sz; j += 2 * nwaves) {
        const int j2 = j + nwaves;
        const int rowA = __builtin_amdgcn_readlane(hdr, __builtin_amdgcn_readfirstlane(j));
        const int rowB = j2 < sz ? __builtin_amdgcn_readlane(hdr, __builtin_amdgcn_readfirstlane(j2)) : -1;
        const bool okA = rowA >= 0 && rowA < a.recv_rows, okB = rowB >= 0 && rowB < a.recv_rows;
        if (!okA || (j2 < sz && !okB)) dev_set_error(a.fifo.error, EP_EBOUNDS);
        const char *srcA = slot + kHtHeader + (size_t)j * rb, *srcB = slot + kHtHeader + (size_t)j2 * rb;
        u32x4 *dstA = (u32x4 *)((char *)a.recv + (size_t)(okA ? rowA : 0) * out_stride);
        u32x4 *dstB = (u32x4 *)((char *)a.recv + (size_t)(okB ? rowB : 0) * out_stride);
        // (the scales behind the codes go to their own array; the first 64 leave with the codes: behind the stores they would wait
        // for those)
        float scaleA = 0.0f, scaleB = 0.0f;
        const int nblk = a.H >> 7;
        if (fp8 && lane < nblk) {
          if (okA) scaleA = __builtin_nontemporal_load((const float *)(srcA + a.H) + lane);
          if (okB) scaleB = __builtin_nontemporal_load((const float *)(srcB + a.H) + lane);
        }
        for (int v0 = lane; v0 < nvec; v0 += 64 * 8) {
          u32x4 ra[8], rb2[8];
          if (okA) ht_load_piece<true, 8>(ra, (const u32x4 *)srcA, v0, nvec);
          if (okB) ht_load_piece<true, 8>(rb2, (const u32x4 *)srcB, v0, nvec);
          if (okA) ht_store_piece<false, 8>(ra, dstA, v0, nvec);
          if (okB) ht_store_piece<false, 8>(rb2, dstB, v0, nvec);
        }
        if (fp8) {
          if (lane < nblk) {
            if (okA) a.recv_scale[(size_t)rowA * nblk + lane] = scaleA;
            if (okB) a.recv_scale[(size_t)rowB * nblk + lane] = scaleB;
          }
          for (int b = lane + 64; b < nblk; b += 64) {
            if (okA) a.recv_scale[(size_t)rowA * nblk + b] = __builtin_nontemporal_load((const float *)(srcA + a.H) + b);
            if (okB) a.recv_scale[(size_t)rowB * nblk + b] = __builtin_nontemporal_load((const float *)(srcB + a.H) + b);
          }
        }
      }
    }
  }
  wait_for_own_stores();  // every load of a slot has returned before the slot is released
  __syncthreads();
  // release the slots: one head Atomic per consumed chunk, numbered on the reverse channel
  const RingDev fifo = ht_fifo();
  for (int r = tid; r < a.R; r += blockDim.x) {
    const int lo = sh.lo[r], hi = sh.hi[r];
    for (int n = lo; n < hi; ++n) {
      const int sz = min(kChunkRows, sh.total[r] - (n << 5));
      ring_push(fifo, (unsigned)(c * a.R + r) % fifo.channels, cmd_w0(EP_OP_RING, a.src, (unsigned)r, (unsigned)c),
                ((unsigned)EP_RING_HEAD << 30) | (unsigned)sz, sh.seqr[r] + (unsigned)n, 0u);
    }
    if (hi > lo) {
      sh.next[r] = hi;
      __hip_atomic_fetch_sub(&sh.remaining, hi - lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      HT_ST(&sh.progress, 1);
    }
  }
}

__global__ __launch_bounds__(1024) void ht_ring_kernel(HtRingArgs a) {
  __shared__ HtShared sh;
  const int tid = threadIdx.x;
  const int c = blockIdx.x;  // the slice
  const int t0 = min(a.T, c * a.slice_len), t1 = min(a.T, t0 + a.slice_len);
  for (int r = tid; r < a.R; r += blockDim.x) {
    sh.total[r] = 0;
    sh.fill[r] = 0;
    sh.seen[r] = 0;
    sh.lock[r] = 0;
    sh.next[r] = 0;
    sh.seqf[r] = a.seq_fwd[c * a.R + r];
    sh.cumf[r] = a.cum_fwd[c * a.R + r];
    sh.seqr[r] = a.seq_rev[c * a.R + r];
    sh.cumr[r] = a.cum_rev[c * a.R + r];
  }
  for (int i = tid; i < a.R * a.W; i += blockDim.x) sh.done[i] = 0;
  if (tid == 0) {
    sh.abort = sh.remaining = sh.progress = sh.idle = sh.announced = 0;
    sh.split = a.split;
  }
  __syncthreads();
  // rows per channel of this slice: both ends count them from the routing table (the count
  // notification that precedes a high-throughput dispatch)
  for (int i = tid; i < (t1 - t0) * a.K; i += blockDim.x) {
    const int e = a.idx[(size_t)t0 * a.K + i], row = a.dst_row[(size_t)t0 * a.K + i];
    if (ht_valid(a, e, row)) {
      __hip_atomic_fetch_add(&sh.total[e / a.E_loc], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    } else if (e >= 0) {
      dev_set_error(a.fifo.error, EP_EBOUNDS);
    }
  }
  __syncthreads();
  ht_share(a, sh, a.split, blockIdx.y);
  __syncthreads();
  if (tid == 0) {
    int chunks = 0;
    for (int r = 0; r < a.R; ++r) chunks += (sh.total[r] + 31) >> 5;
    sh.remaining = chunks;
  }
  __syncthreads();

  int q = 0;  // this wave has sent its first q tokens
  HtToken tk{0ull, 0};
  bool sent_all = false;
  unsigned long long last = wall_clock64();
  while (HT_LD(&sh.remaining) > 0) {  // (uniform: read between two barriers that no writer crosses)
    if (!sent_all) sent_all = ht_send_step(a, sh, c, t0, t1 - t0, q, tk);
    __syncthreads();
    ht_receive_step(a, sh, c);
    __syncthreads();
    if (tid == 0) {
      const unsigned long long now = wall_clock64();
      const int progressed = HT_LD(&sh.progress);
      sh.idle = !progressed;
      if (progressed) {
        last = now;
        sh.progress = 0;
      } else if (now - last > a.fifo.timeout_ticks) {
        dev_set_error(a.fifo.error, EP_ETIMEOUT);
        sh.abort = 1;
      }
    }
    __syncthreads();
    if (sh.abort) break;
    if (sh.idle) __builtin_amdgcn_s_sleep(127);
  }
  __syncthreads();
  // the channels' running sequence numbers and row totals, for the next dispatch
  for (int r = tid; r < a.R; r += blockDim.x) {
    if (!sh.mine[r]) continue;
    const unsigned nch = (unsigned)(sh.total[r] + 31) >> 5;
    a.seq_fwd[c * a.R + r] = sh.seqf[r] + 2u * nch;
    a.cum_fwd[c * a.R + r] = sh.cumf[r] + (unsigned)sh.total[r];
    a.seq_rev[c * a.R + r] = sh.seqr[r] + nch;
    a.cum_rev[c * a.R + r] = sh.cumr[r] + (unsigned)sh.total[r];
  }
  drain_all_channels(ht_fifo(), a.waves_done, (unsigned)a.src, lane_id());
}
static_assert(std::is_same_v<decltype(&ht_ring_kernel), void (*)(HtRingArgs)> && std::is_standard_layout_v<HtRingArgs>,
              "ht_fifo takes the kernel's arguments for one HtRingArgs");

// A workgroup's sixteen waves fill a compute unit, so fewer than 256 slices leave some idle: then 2, 4, ... workgroups share a
// slice, up to the number of ranks, each with the channels that ht_share deals to it (a channel's state is its own, so they
// have nothing to say to each other).  As long as each still has half a megabyte to move; with less, the polls and the reads
// of the tokens, which every one of them does, cost more.  Whole steps, 1 / 2 / 4 / 8 / 16 workgroups a slice, us, taken with every
// workgroup at every 2nd, 4th, ... rank and an acquire by every wave (now 128 slices, 4096 x 7168 400, 64 slices, 1500 x 7168 163):
//   4 slices    4096 tokens x 7168 top-8 4783 / 3045 / 2662 / 2344 / 2415, 1024 x 7168 1151 / 780 / 683 / 515 / 404, 4096 x
//               2048 1831 / 1402 / 1422 / 1486 / 1704 (16 by this rule: rows this narrow would be better off with 2)
//   8 slices    4096 x 7168 2536 / 1610 / 1396 / 1234 / 1174, 4096 x 2048 972 / 713 / 732 / 755 / 787
//   16 slices   4096 x 7168 1435 / 1003 / 873 / 698 / 631, 1024 x 7168 332 / 234 / 202 / 169 / 161 (0.46 MB each)
//   64 slices   4096 tokens x 7168 top-8 656 / 514 / 441, 1536 x 7168 265 / 223 / 218, 1024 x 7168 179 / 170 / 168 (0.46 MB
//               each), 768 x 7168 141 / 138 / 148 (0.34 MB), 1024 x 4096 113 / 109 / 127 (0.26 MB), in FP8 101 / 104 (0.27
//               MB) / 129, 2048 x 2048 125 / 124 / 143 (0.26 MB)
//   128 slices  4096 x 7168 474 / 439, 2048 x 7168 top-6 211 / 202, 4096 x 4096 in FP8 242 / 240, 1024 x 7168 188 / 194 (0.46
//               MB), 1536 x 2048 in FP8 121 / 148 (0.1 MB)
constexpr long long kHtSplitBytes = 500000;
int launch_ht_ring(const HtRingArgs &a, const Tunables &tune, void *stream) {
  int threads = tune.ht_threads;
  if (threads < 64 || threads > 1024 || (threads & 63)) threads = 1024;
  HtRingArgs b = a;
  const long long bytes = (long long)a.T * a.K * a.row_bytes;
  b.split = 1;
  while (b.split * 2 <= a.R && b.split * 2 * a.slices <= 256 && bytes >= kHtSplitBytes * a.slices * b.split * 2) b.split *= 2;
  hipLaunchKernelGGL(ht_ring_kernel, dim3((unsigned)b.slices, (unsigned)b.split), dim3((unsigned)threads), 0,
                     (hipStream_t)stream, b);
  return (int)hipGetLastError();
}

}  // namespace ep
