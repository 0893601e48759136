// Dispatch (bf16 / FP8 E4M3) and the emission of transfer commands: HBM-bound row copies with 16-byte vector
// accesses, one wavefront per token or per slice of a token; no dense contraction, hence no MFMA.
#include "ep_device.h"

namespace ep {

// ------------------------------------------------- dispatch: command emission
struct TokenMeta {
  int e;       // expert of this lane's k (lane < K), -1 otherwise
  int row;     // destination row
  bool valid;  // this (t, k) is dispatched by this call
};

// Which group of tokens this workgroup takes: launch order, or the mirror image of it.
EP_DEV int token_block(const DispatchArgs &a) {
  return a.reverse ? (int)gridDim.x - 1 - (int)blockIdx.x : (int)blockIdx.x;
}

EP_DEV TokenMeta load_meta(const DispatchArgs &a, int t, int lane) {
  TokenMeta m{-1, -1, false};
  if (t < a.T && lane < a.K) {
    m.e = a.idx[(size_t)t * a.K + lane];
    m.row = a.dst_row[(size_t)t * a.K + lane];
    if (m.e >= 0) {
      if (m.e >= a.E || m.row < 0 || m.row >= a.recv_rows)
        dev_set_error(a.ring.error, EP_EBOUNDS);
      else if (a.filter < 0 || m.e / a.E_loc == a.filter)
        m.valid = true;
    } else if (m.e != -1) {
      dev_set_error(a.ring.error, EP_EBOUNDS);
    }
  }
  return m;
}

EP_DEV void push_count_atomic(const DispatchArgs &a, int e, int value) {
  const unsigned dr = (unsigned)(e / a.E_loc), le = (unsigned)(e - (int)dr * a.E_loc);
  ring_push(a.ring, (unsigned)e % a.ring.channels, cmd_w0(EP_OP_ATOMIC, a.src, dr, le), (unsigned)value, 0u,
            (unsigned)(a.src * a.E_loc) + le);
}

// The same by a whole wave, for the lanes with `push`.
EP_DEV void push_count_atomics(const DispatchArgs &a, bool push, int e, int value, u32x4 *scratch) {
  if (!push) e = 0;
  const unsigned dr = (unsigned)(e / a.E_loc), le = (unsigned)(e - (int)dr * a.E_loc);
  ring_push_sorted(a.ring, push, (unsigned)e % a.ring.channels, cmd_w0(EP_OP_ATOMIC, a.src, dr, le), (unsigned)value, 0u,
                   (unsigned)(a.src * a.E_loc) + le, scratch);
}

// Workgroup 0, ahead of its rows: the count Atomics that no row completion will trigger - experts with count 0, or all of
// them when the caller wants the atomics ahead of the writes.  With one command per row the wave that pushes for the group
// has no part in it: up to kLeadWaves others take 64 experts each at a time.
constexpr int kLeadWaves = 4;
template <bool GROUPS>
EP_DEV void emit_leading_atomics(const DispatchArgs &a, int wave, int lane) {
  extern __shared__ u32x4 s_dyn[];  // (one command per row: the scratch of ring_push_sorted for waves 0 to kLeadWaves)
  const bool first = (a.cmd_mode & EP_CMD_ATOMICS_FIRST) != 0;
  const int waves = GROUPS ? min(kLeadWaves, (int)(blockDim.x >> 6) - 1) : 1, w = GROUPS ? wave - 1 : wave;
  if (w < 0 || w >= waves) return;
  for (int e0 = w * 64; e0 < a.E; e0 += waves * 64) {
    const int e = e0 + lane;
    const int c = e < a.E ? a.count[e] : -1;
    const bool push = c >= 0 && (first || c == 0) && (a.filter < 0 || e / a.E_loc == a.filter);
    if (GROUPS)
      push_count_atomics(a, push, e, c, s_dyn + wave * (kSortScratch / 16));
    else if (push)
      push_count_atomic(a, e, c);
  }
}

// The chunk modes' commands (one Write per row: emit_group_cmds).  Called by a whole wave, whose valid lanes hold a dispatched
// (t,k) each, after the token's rows are stored and acknowledged (write-through, so they are in memory).  The lane that
// completes a run of <= 32 consecutive rows of an expert pushes the Write for the run.  Whoever completes the expert pushes its
// count Atomic (Section 3.3: the receiver holds it until that many rows arrived).  The scratch counters return to zero by
// themselves.
EP_DEV void emit_chunk_cmds(const DispatchArgs &a, const TokenMeta &m) {
  const int e = m.valid ? m.e : 0;
  const unsigned dr = (unsigned)(e / a.E_loc), le = (unsigned)(e - (int)dr * a.E_loc);
  const int mode = a.cmd_mode & EP_CMD_MODE_MASK;
  int c = 0, csize = 0;
  unsigned len = 0, off16 = 0;
  bool whole = false;  // this lane's row was the last one of its chunk
  if (m.valid) {
    c = a.count[e];
    const int base = a.base[e], slot = m.row - base, j = slot >> 5;
    if (slot < 0 || j >= a.chunks_per_expert || slot >= c) {
      dev_set_error(a.ring.error, EP_EBOUNDS);
    } else {
      csize = min(kChunkRows, c - (j << 5));
      len = (unsigned)csize * a.row_bytes;
      off16 = (unsigned)(((unsigned long long)(base + (j << 5)) * a.row_bytes) >> 4);
      int *cnt = a.chunk_cnt + (size_t)e * a.chunks_per_expert + j;
      whole = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == csize;
      if (whole) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (__ballot(whole) == 0ull) return;
  if (mode == EP_CMD_CHUNK32_ORDERED) {
    // High-throughput style: the chunk's Write and the Atomic that advances the receiver's tail
    // take two consecutive sequence numbers of the communication channel (source, destination
    // rank) and travel through that channel's FIFO; the receiver re-establishes the order.
    unsigned seq = 0;
    if (whole)
      seq = __hip_atomic_fetch_add(a.ht_seq + (size_t)a.src * a.R + dr, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ring_push_pairs(a.ring, whole, dr % a.ring.channels,
                    u32x4{cmd_w0(EP_OP_ORDERED_WRITE, a.src, dr, le), ((unsigned)(csize - 1) << 26) | (len >> 4), seq, off16},
                    u32x4{cmd_w0(EP_OP_ORDERED_ATOMIC, a.src, dr, 0), (unsigned)csize, seq + 1u, (unsigned)(a.src * a.R) + dr});
    return;
  }
  if (whole) {
    // Everything for one destination expert goes through one FIFO (and therefore one proxy thread):
    // in-FIFO order is the only order the channel guarantees (Section 3.1, "GPU-side contention").
    const unsigned ch = (unsigned)e % a.ring.channels;
    unsigned long long idx = __hip_atomic_fetch_add(&a.ring.tail[ch], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Counted once the Write has its Idx, so that the expert's Atomic, whoever pushes it, gets a later one; together with
    // the read of the head.  (4096 tokens x 7168 109.2 us, the head first and then the count 110.2; 2048 x 2048 10.7 and 11.2.)
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(idx) : : "memory");
    const int done =
        __hip_atomic_fetch_add(a.expert_done + e, csize, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + csize;
    ring_publish(a.ring, ch, idx, cmd_w0(EP_OP_WRITE, a.src, dr, le), ((unsigned)(csize - 1) << 26) | (len >> 4), off16,
                 off16);
    if (done == c) {
      __hip_atomic_store(a.expert_done + e, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!(a.cmd_mode & EP_CMD_ATOMICS_FIRST)) push_count_atomic(a, e, c);
    }
  }
}

// One command per row: a group of workgroups holds about 64 (token, k) pairs, and the first wave of the group's last
// workgroup to store its rows pushes for all of them, sorted by channel, so that the commands of a channel leave as one
// run of consecutive slots written by neighbouring lanes (see ring_push_sorted).  The groups' counters are
// their own (a table may be dispatched in parts, which leaves chunk counters half way between two calls) and return to
// zero by themselves.
// What a small dispatch waits for is the proxy, which misses its caches once for every write that reaches a polled line.
// Whole steps, groups / every workgroup on its own (us, rows of 7168, top-8 of 256 experts): 128 tokens 30 / 36, 256: 34 /
// 51, 512: 48 / 73; 512 tokens x 4096: 41 / 49.
// Bound by the chain of round trips behind the last row: the group's counter, the pairs, the reservation, the experts'
// counters, the cached heads, and for complete experts a reservation and the heads once more.  The experts are counted ahead
// of the command stores: behind them, the wait for the counters is one for the host's acknowledgement of the stores as well.
// Whole steps, counted behind the stores / ahead of them, us: 8192 tokens x 1024 top-4 of 128 experts 109 / 83, of 256 112 /
// 94, 4096 x 7168 top-8 in FP8 178 / 177.  With the leading Atomics pushed by the same wave ahead of its row (64 experts after
// the other) one token of 256 experts, alone, takes 35 us, now 33; larger steps are the same.  With the pairs loaded ahead of
// the rows, which then wait for them too, 8192 x 1024 took 14 us more; with the leading Atomics in a workgroup of their own,
// where the proxy sees them first, 128 tokens 1 us more.
// Where a workgroup pushes its own, the heads are read ahead (ring_refresh_ahead) up to the last quarter of the grid.  Whole steps,
// without / with, us: 8192 tokens x 4096 top-8 247 / 240, in FP8 232 / 219, 4096 x 7168 205 / 203, 2048 x 7168 112 / 108; rings of
// 2048 265 / 243; 16 channels 250 / 239; up to seven eighths of the grid the first 237, the last but two 109, with 16 channels
// 243.  With 32 channels, which all come to the same place in their rings at once, 272 / 271, 230 / 236 and in FP8 248 / 258:
// not there.  Small dispatches fill a ring once in thirty steps.
constexpr unsigned kRefreshChannels = 16;
EP_DEV void emit_group_cmds(const DispatchArgs &a, int wave, int lane) {
  extern __shared__ u32x4 s_dyn[];  // the scratch of ring_push_sorted
  __syncthreads();  // every wave has waited for its own stores before it came here
  if (wave != 0) return;
  const int gb = a.blocks_per_group, group = token_block(a) / gb;
  if (gb > 1) {
    int last = 0;
    if (lane == 0) {
      int *cnt = a.group_cnt + group;
      last = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
             min(gb, (int)gridDim.x - group * gb);
      if (last) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!__builtin_amdgcn_readfirstlane(last)) return;
  }
  const int tokens = gb * a.tokens_per_block, t0 = group * tokens, n = min(tokens, a.T - t0) * a.K;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + lane;
    int e = -1, row = -1;
    if (i < n) {
      e = a.idx[(size_t)t0 * a.K + i];
      row = a.dst_row[(size_t)t0 * a.K + i];
    }
    // (an entry out of range has been reported by its own wave)
    const bool active = e >= 0 && e < a.E && row >= 0 && row < a.recv_rows && (a.filter < 0 || e / a.E_loc == a.filter);
    if (!active) e = 0;
    const int c = a.count[e];
    const unsigned dr = (unsigned)(e / a.E_loc), le = (unsigned)(e - (int)dr * a.E_loc), ch = (unsigned)e % a.ring.channels;
    const unsigned long long so = (unsigned long long)(t0 + i / a.K) * a.row_bytes;
    const unsigned long long dof = (unsigned long long)row * a.row_bytes;
    SortedRun run = ring_reserve_sorted(a.ring, active, ch);
    // Counted once the Writes have their Idx: an expert's Atomic, whoever pushes it, gets a later one.
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(run.idx) : : "memory");
    int done = 0;
    if (active) done = __hip_atomic_fetch_add(a.expert_done + e, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ring_publish_sorted(a.ring, active, run, ch, cmd_w0(EP_OP_WRITE, a.src, dr, le), a.row_bytes >> 4, (unsigned)(so >> 4),
                        (unsigned)(dof >> 4), s_dyn);
    const bool complete = active && done + 1 == c;
    if (complete) __hip_atomic_store(a.expert_done + e, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    push_count_atomics(a, complete && !(a.cmd_mode & EP_CMD_ATOMICS_FIRST), e, c, s_dyn);
    if (gb == 1 && a.ring.channels <= kRefreshChannels && blockIdx.x < gridDim.x / 4 * 3)
      ring_refresh_ahead(a.ring, active, ch, run.idx);
  }
}

EP_DEV void emit_drain(const DispatchArgs &a, int lane) {
  drain_all_channels(a.ring, a.waves_done, (unsigned)a.src, lane);
}

// ------------------------------------------------------------ dispatch bf16
// A token's row is H/8 16-byte vectors.  Wavefront (token, part) reads its
// slice of the row ONCE into registers (VPL vectors per lane) and stores it to
// every destination row; destination rows are wave-uniform and come from the
// lanes that hold the token's (expert, row) pairs.
// (A row's stores wait for those of the wave's row before.  Left to the compiler, which has to wait for the loads somewhere,
// the wait is before every row, every store or the first row only, as the register allocation falls.  Before every row is
// best on the whole, us: ring off 8192 tokens x 4096 112, without waits 119; 1536 x 12288 47 and 52; one command per row 1536
// x 9216 54 and 52, with a wait before every store 64.)
// (GROUPS: one command per row.  Instances of their own keep both at or below 98 scalar registers, by the compiler's count
// eight waves per SIMD; together they take 103 to 105, seven waves: 1536 x 16384, 16 waves per workgroup, 94 us, apart 90.)
// (The row leaves for the registers ahead of the token's pairs, which say where it goes: one round trip instead of two before a
// wave's first store.  Pairs first / together, whole steps, us: 4096 tokens x 7168 top-8 with chunks 197.3 / 195.2, in FP8
// 164.4 / 163.2, deduplicated over 16 groups 357.3 / 352.4; 420 x 7552 in FP8 33.6 / 32.9.  With one command per row, where a
// workgroup has its pairs to push and waits for them anyway, the pairs stay first: 8192 x 4096 249 / 257.  So they do for
// sequenced chunks (1531 x 5120 top-6 57.6 / 59.6; with the choice made in the kernel 59), for one rank of several, whose rows
// are a few tokens' only, and with more than four vectors per lane, for which it was not measured.)
// (Write-through stores without the streaming hint: with it the dispatch itself and a combine of other rows are up to 4%
// faster, but whoever reads the rows next no longer finds any in the memory-side cache.  Step and a read of the received
// rows, without / with, us: 4058 tokens x 7168 top-8 in FP8 182 / 194, 8116 tokens 365 / 380, 8239 x 4096 bf16 337 / 341.)
// (The same placement as in dispatch_bf16_kernel below, as a function for the form with a command wave; the plain
// kernel keeps its own copy: with the body moved into a function the compiler allocated 61 instead of 46
// registers for it and spilled at 7 and 8 vectors per lane.)
template <int VPL>
EP_DEV void place_token_bf16(const DispatchArgs &a, const int row_of_lane, unsigned long long vmask, int t, int part,
                             int lane) {
  if (!vmask || (a.cmd_mode & EP_CMD_NO_PLACEMENT)) return;
  const int nvec = a.H >> 3;
  const int v0 = part * VPL * 64 + lane;
  const u32x4 *src = (const u32x4 *)a.x + (size_t)t * nvec;
  u32x4 v[VPL];
#pragma unroll
  for (int i = 0; i < VPL; ++i)
    if (v0 + i * 64 < nvec) v[i] = __builtin_nontemporal_load(src + v0 + i * 64);
  unsigned long long mm = vmask;
  while (mm) {
    const int k = __builtin_ctzll(mm);
    mm &= mm - 1;
    const int row = __builtin_amdgcn_readlane(row_of_lane, k);
    u32x4 *dst = (u32x4 *)a.recv + (size_t)row * nvec;
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (v0 + i * 64 < nvec) store_payload(dst + v0 + i * 64, v[i]);
  }
}

// A token without any expert (padding) has a row that nobody wants: the first of its pairs tells, a scalar load that the row
// then waits for.  (A token whose first pair was dropped reads its row behind its pairs.)  Ring off, pairs first / every row
// ahead / this, us: 4096 tokens x 7168 top-8 102.8 / 100.0 / 102.4, with every fifth token dropped 85.4 / 82.0 / 83.6, half of
// them 64.9 / 58.9 / 62.4, 19 of 20 16.4 / 24.3 / 18.1; 16000 x 1024 48.3 / 45.2 / 45.0, 38.2 / 41.0 / 32.0, 20.7 / 32.7 /
// 20.7, 8.5 / 10.2 / 9.2; 4096 x 7168 in FP8 56.4 / 52.9 / 51.4, 54.5 / 45.3 / 48.5, 33.6 / 35.3 / 30.6, 7.0 / 14.8 / 7.9; 2000
// x 7168 in FP8 25.8 / 23.9 / 23.8, 19.2 / 20.5 / 19.1, 12.9 / 16.3 / 13.4, 5.2 / 7.7 / 5.4.
EP_DEV bool names_an_expert(const DispatchArgs &a, int t) { return t < a.T && a.idx[(size_t)t * a.K] >= 0; }

// Which rows leave ahead of their pairs: none, every one, or those of tokens that name an expert.
enum { kAheadNone = 0, kAheadAll = 1, kAheadNamed = 2 };

template <int VPL, bool GROUPS, int AHEAD>
__global__ void dispatch_bf16_kernel(DispatchArgs a) {
  const int wave = wave_id(), lane = lane_id();
  const int part = (unsigned)wave % (unsigned)a.parts;
  const int t = token_block(a) * a.tokens_per_block + (unsigned)wave / (unsigned)a.parts;
  const bool ring_on = (a.cmd_mode & EP_CMD_MODE_MASK) != EP_CMD_NONE;
  const bool ordered = (a.cmd_mode & EP_CMD_MODE_MASK) == EP_CMD_CHUNK32_ORDERED;
  const bool ahead = AHEAD == kAheadNamed ? names_an_expert(a, t) : AHEAD == kAheadAll && t < a.T;
  if (ring_on && !ordered && blockIdx.x == 0) emit_leading_atomics<GROUPS>(a, wave, lane);

  const int nvec = a.H >> 3;
  const int v0 = part * VPL * 64 + lane;
  const u32x4 *src = (const u32x4 *)a.x + (size_t)t * nvec;
  u32x4 v[VPL];
  auto load = [&]() {
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (v0 + i * 64 < nvec) v[i] = __builtin_nontemporal_load(src + v0 + i * 64);
  };
  if (ahead) load();
  const TokenMeta m = load_meta(a, t, lane);
  unsigned long long vmask = __ballot(m.valid);
  if (vmask && !(a.cmd_mode & EP_CMD_NO_PLACEMENT)) {
    if (AHEAD != kAheadAll && !ahead) load();
    unsigned long long mm = vmask;
    while (mm) {
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      const int k = __builtin_ctzll(mm);
      mm &= mm - 1;
      const int row = __builtin_amdgcn_readlane(m.row, k);
      u32x4 *dst = (u32x4 *)a.recv + (size_t)row * nvec;
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (v0 + i * 64 < nvec) store_payload(dst + v0 + i * 64, v[i]);
    }
  }
  if (!ring_on) return;
  wait_for_own_stores();  // the rows are in memory before a counter or command mentions them
  if constexpr (GROUPS) {
    emit_group_cmds(a, wave, lane);
  } else {
    if (a.parts > 1) __syncthreads();
    if (part == 0) emit_chunk_cmds(a, m);
  }
  if (a.cmd_mode & EP_CMD_DRAIN) emit_drain(a, lane);
}

// ------------------------------------------------------------- dispatch FP8
template <int VPL>
EP_DEV void place_token_fp8(const DispatchArgs &a, const TokenMeta &m, unsigned long long vmask, int t, int part) {
  if (!vmask) return;
  const int lane = lane_id();
  const int npair = a.H >> 4;  // 16-channel groups per row
  const int nblk = a.H >> 7;   // 128-channel blocks per row
  const int p0 = part * VPL * 64 + lane;
  {
    const u32x4 *src = (const u32x4 *)a.x + (size_t)t * npair * 2;
    u32x4 lo[VPL], hi[VPL], q[VPL];
    float sc[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (p0 + i * 64 < npair) {
        lo[i] = __builtin_nontemporal_load(src + 2 * (p0 + i * 64));
        hi[i] = __builtin_nontemporal_load(src + 2 * (p0 + i * 64) + 1);
      } else {
        lo[i] = u32x4{0, 0, 0, 0};
        hi[i] = u32x4{0, 0, 0, 0};
      }
#pragma unroll
    for (int i = 0; i < VPL; ++i) quant16(lo[i], hi[i], q[i], sc[i]);
    // Where a row goes: into the two receive arrays (codes, scales), or - when the proxy moves the rows -
    // as ONE message of row_bytes bytes (the H codes, then the H/128 fp32 scales, padded to 16 bytes:
    // the ~7 KB token of Section 2.1) into the send heap: at its destination row for chunk commands
    // (the heap mirrors the receive heap), or once, at the token's own row, for per-token commands.
    unsigned long long mm = a.msg_rows == 2 ? 1ull : vmask;
    while (mm) {
      const int k = __builtin_ctzll(mm);
      mm &= mm - 1;
      const int row = a.msg_rows == 2 ? t : __builtin_amdgcn_readlane(m.row, k);
      u32x4 *dq;
      float *ds;
      if (a.msg_rows) {
        char *msg = (char *)a.recv + (size_t)row * a.row_bytes;
        dq = (u32x4 *)msg;
        ds = (float *)(msg + a.H);
      } else {
        dq = (u32x4 *)a.recv + (size_t)row * npair;
        ds = a.recv_scale + (size_t)row * nblk;
      }
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (p0 + i * 64 < npair) {
          store_payload(dq + p0 + i * 64, q[i]);
          if ((lane & 7) == 0)
            __hip_atomic_store(ds + ((p0 + i * 64) >> 3), sc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
  }
}

// (TOGETHER: a row's scales leave as one store, by one wave, out of LDS; else every wave stores those of its part, 32 bytes at
// a time.  Each store that fills no line of its own costs the memory behind the L2 as much as a full one, and there are seven
// of them beside the 56 lines of a 7168-wide row's codes; where the rows fit the memory-side cache (256 MB) beside what else is
// in it, the barrier costs more.  Whole steps, apart / together, us: 4096 tokens x 7168 top-8 (242 MB) 163.8 / 161.3, with a
// tenth of the pairs dropped 152.6 / 152.1, three tenths 127.7 / 129.3; 12000 x 2048 (203 MB) 156.6 / 153.6, 142.7 / 145.1,
// 121.3 / 123.5; 6000 x 4096 (203 MB) 138.6 / 136.7, 125.9 / 127.2, 102.7 / 103.7; 3000 x 7168 (177 MB) 118.6 / 122.2, 2700 x
// 8192 122.6 / 123.3, 6000 x 3072 102.1 / 105.3, 8192 x 2048 97.2 / 97.9.  A row that is one wave's has one store of scales
// anyway: ring off, 30000 x 1024 49.7 / 51.8.  With one command per row it was not measured.)
// (AHEAD: the row leaves together with the pairs, see dispatch_bf16_kernel, but for sequenced chunks: that choice is made here,
// as with instances of their own those got slower, 2000 tokens x 7168 top-8 89.8 us, apart 93.9, 4096 tokens 167.8, 169.7.  For
// one rank of several, whose launches are small, an instance without: ring off, one of 16 ranks, 4096 x 7168 10.6 us, apart
// 10.2.)
template <int VPL, bool GROUPS, bool AHEAD, bool TOGETHER>
__global__ void dispatch_fp8_kernel(DispatchArgs a) {
  __shared__ float s_scale[TOGETHER ? 16 * VPL * 8 : 1];  // [wave][its blocks]: the parts of a token in a row
  const int wave = wave_id(), lane = lane_id();
  const int part = (unsigned)wave % (unsigned)a.parts;
  const int t = token_block(a) * a.tokens_per_block + (unsigned)wave / (unsigned)a.parts;
  const bool ring_on = (a.cmd_mode & EP_CMD_MODE_MASK) != EP_CMD_NONE;
  const bool ordered = (a.cmd_mode & EP_CMD_MODE_MASK) == EP_CMD_CHUNK32_ORDERED;
  const bool ahead = AHEAD && !ordered && names_an_expert(a, t);
  if (ring_on && !ordered && blockIdx.x == 0) emit_leading_atomics<GROUPS>(a, wave, lane);

  const int npair = a.H >> 4;  // 16-channel groups per row
  const int nblk = a.H >> 7;   // 128-channel blocks per row
  const int p0 = part * VPL * 64 + lane;
  const u32x4 *src = (const u32x4 *)a.x + (size_t)t * npair * 2;
  u32x4 lo[VPL], hi[VPL], q[VPL];
  float sc[VPL];
  auto load = [&]() {
#pragma unroll
    for (int i = 0; i < VPL; ++i)
      if (p0 + i * 64 < npair) {
        lo[i] = __builtin_nontemporal_load(src + 2 * (p0 + i * 64));
        hi[i] = __builtin_nontemporal_load(src + 2 * (p0 + i * 64) + 1);
      } else {
        lo[i] = u32x4{0, 0, 0, 0};
        hi[i] = u32x4{0, 0, 0, 0};
      }
  };
  if (ahead) load();
  const TokenMeta m = load_meta(a, t, lane);
  unsigned long long vmask = __ballot(m.valid);
  if (vmask) {
    if (!ahead) load();
#pragma unroll
    for (int i = 0; i < VPL; ++i) quant16(lo[i], hi[i], q[i], sc[i]);
    if (TOGETHER && (lane & 7) == 0)
#pragma unroll
      for (int i = 0; i < VPL; ++i) s_scale[(wave * VPL + i) * 8 + (lane >> 3)] = sc[i];
    // Where a row goes: into the two receive arrays (codes, scales), or - when the proxy moves the rows -
    // as ONE message of row_bytes bytes (the H codes, then the H/128 fp32 scales, padded to 16 bytes:
    // the ~7 KB token of Section 2.1) into the send heap: at its destination row for chunk commands
    // (the heap mirrors the receive heap), or once, at the token's own row, for per-token commands.
    unsigned long long mm = a.msg_rows == 2 ? 1ull : vmask;
    while (mm) {
      const int k = __builtin_ctzll(mm);
      mm &= mm - 1;
      const int row = a.msg_rows == 2 ? t : __builtin_amdgcn_readlane(m.row, k);
      u32x4 *dq;
      float *ds;
      if (a.msg_rows) {
        char *msg = (char *)a.recv + (size_t)row * a.row_bytes;
        dq = (u32x4 *)msg;
        ds = (float *)(msg + a.H);
      } else {
        dq = (u32x4 *)a.recv + (size_t)row * npair;
        ds = a.recv_scale + (size_t)row * nblk;
      }
#pragma unroll
      for (int i = 0; i < VPL; ++i)
        if (p0 + i * 64 < npair) {
          store_payload(dq + p0 + i * 64, q[i]);
          if (!TOGETHER && (lane & 7) == 0)
            __hip_atomic_store(ds + ((p0 + i * 64) >> 3), sc[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
  }
  if constexpr (TOGETHER) {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // (the codes' stores are not waited for)
    const float *scales = s_scale + (wave - part) * VPL * 8;
    int n = 0;
    for (unsigned long long mm = vmask; mm; mm &= mm - 1, ++n) {
      if (n % a.parts != part) continue;  // the token's waves take its rows in turns
      const int row = __builtin_amdgcn_readlane(m.row, __builtin_ctzll(mm));
      float *ds = a.msg_rows ? (float *)((char *)a.recv + (size_t)row * a.row_bytes + a.H) : a.recv_scale + (size_t)row * nblk;
      for (int b = lane; b < nblk; b += 64) __hip_atomic_store(ds + b, scales[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  if (!ring_on) return;
  wait_for_own_stores();
  if constexpr (GROUPS) {
    emit_group_cmds(a, wave, lane);
  } else {
    if (a.parts > 1) __syncthreads();
    if (part == 0) emit_chunk_cmds(a, m);
  }
  if (a.cmd_mode & EP_CMD_DRAIN) emit_drain(a, lane);
}

// ------------------------------------------- dispatch with a command wavefront
// Ring-on launches: persistent workgroups of D data waves and ONE command wave.  A data wave places its
// slice of a token, waits for its own stores, leaves the token's (expert, row) pairs in LDS and goes on
// to the workgroup's next batch of tokens; the command wave picks the batch up when all D waves have
// signed it off and does everything that needs a round trip through the L2 or a store to host memory -
// completion counting, Idx reservation, the Push itself, count Atomics - while the data waves are already
// storing the next batch.  Two batches of pairs fit the LDS, so the command wave may lag one batch behind.
// Waits between the waves are LDS polls, each bounded by the ring's time limit.
// Selected with EP_DISPATCH_PIPELINE=1 and off by default: measured on MI355X (4096 tokens x 7168, and 8192 x
// 4096) it is no faster than the plain form with chunk commands (111.9 vs 112.2 us, 125.6 vs 123.7 us) and
// slower with one command per row (121.8 vs 116.0 us, 158.9 vs 146.2 us).  Under a saturating store stream
// every round trip of the command wave (Idx reservation, head check, completion counting) queues behind the
// compute unit's own stores and takes microseconds, so one command wave per workgroup falls behind its data
// waves; and the row stores themselves run at the rate the memory system gives scattered rows whatever the
// kernel's shape, so hiding the commands' latency buys nothing there.
EP_DEV void pipe_wait_at_least(int *p, int want, const RingDev &r) {
  if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= want) return;
  const unsigned long long t0 = wall_clock64();
  while (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < want) {
    if (wall_clock64() - t0 > r.timeout_ticks) {
      dev_set_error(r.error, EP_ETIMEOUT);
      break;
    }
    __builtin_amdgcn_s_sleep(2);
  }
}

template <int VPL, bool FP8>
__global__ __launch_bounds__(1024) void dispatch_pipelined_kernel(DispatchArgs a) {
  extern __shared__ u32x4 s_dyn[];
  int *ctl = (int *)s_dyn;  // [0], [1]: sign-offs per slot (running totals); [2]: batches the command wave is through
  const int tpb = a.tokens_per_block, n = tpb * a.K, npad = (n + 1) & ~1;
  int2 *pairs = (int2 *)(ctl + 4);               // [2][npad]
  u32x4 *scratch = (u32x4 *)(pairs + 2 * npad);  // 2 KB for ring_push_sorted
  const int wave = threadIdx.x >> 6, lane = lane_id();
  const int D = a.parts * tpb;
  const int nb = (a.T + tpb - 1) / tpb;
  const int mode = a.cmd_mode & EP_CMD_MODE_MASK;
  if (threadIdx.x < 4) ctl[threadIdx.x] = 0;
  __syncthreads();
  if (wave < D) {
    const int part = wave % a.parts, tok = wave / a.parts;
    int it = 0;
#pragma nounroll
    for (int b = blockIdx.x; b < nb; b += gridDim.x, ++it) {
      const int t = (a.reverse ? nb - 1 - b : b) * tpb + tok;
      const TokenMeta m = load_meta(a, t, lane);
      const unsigned long long vmask = __ballot(m.valid);
      if (FP8) place_token_fp8<VPL>(a, m, vmask, t, part);
      else place_token_bf16<VPL>(a, m.row, vmask, t, part, lane);
      wait_for_own_stores();  // the rows are in memory before a counter or command mentions them
      const int slot = it & 1;
      if (it >= 2) pipe_wait_at_least(&ctl[2], it - 1, a.ring);  // the batch that used this slot last is through
      if (part == 0 && lane < a.K) pairs[slot * npad + tok * a.K + lane] = make_int2(m.valid ? m.e : -1, m.row);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      if (lane == 0) __hip_atomic_fetch_add(&ctl[slot], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  } else {
    if (mode != EP_CMD_CHUNK32_ORDERED && blockIdx.x == 0) emit_leading_atomics<false>(a, 0, lane);
    int it = 0;
#pragma nounroll
    for (int b = blockIdx.x; b < nb; b += gridDim.x, ++it) {
      const int t0 = (a.reverse ? nb - 1 - b : b) * tpb;
      const int slot = it & 1;
      pipe_wait_at_least(&ctl[slot], D * (it / 2 + 1), a.ring);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      const int2 *pp = pairs + slot * npad;
      for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        const int2 p = i < n ? pp[i] : make_int2(-1, -1);
        const bool active = p.x >= 0;
        const int t = t0 + i / a.K;
        if (mode == EP_CMD_PER_TOKEN) {  // one command per row, sorted by channel (see ring_push_sorted)
          const int e = active ? p.x : 0;
          const unsigned dr = (unsigned)(e / a.E_loc), le = (unsigned)(e - (int)dr * a.E_loc);
          const unsigned long long so = (unsigned long long)t * a.row_bytes;
          const unsigned long long dof = (unsigned long long)p.y * a.row_bytes;
          ring_push_sorted(a.ring, active, (unsigned)e % a.ring.channels, cmd_w0(EP_OP_WRITE, a.src, dr, le),
                           a.row_bytes >> 4, (unsigned)(so >> 4), (unsigned)(dof >> 4), scratch);
          if (active) {
            const int c = a.count[e];
            if (__hip_atomic_fetch_add(a.expert_done + e, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == c) {
              __hip_atomic_store(a.expert_done + e, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              if (!(a.cmd_mode & EP_CMD_ATOMICS_FIRST)) push_count_atomic(a, e, c);
            }
          }
        } else {
          emit_chunk_cmds(a, TokenMeta{p.x, p.y, active});
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // the pairs have been read: the slot may be refilled
      if (lane == 0) __hip_atomic_store(&ctl[2], it + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  if (a.cmd_mode & EP_CMD_DRAIN) emit_drain(a, lane);
}

// units = 16-byte vectors (bf16) or 16-channel groups (FP8) per row; returns how many of them one
// lane carries.  The row then takes ceil(units / (64 * result)) waves, at most 16.
static int split_for(int units, int T, const int *cands, int ncand) {
  int best = cands[ncand - 1];
  for (int i = 0; i < ncand; ++i)
    if (cands[i] * 256 >= units) {
      best = cands[i];
      break;
    }
  for (int i = ncand - 1; i >= 0; --i) {
    if (cands[i] >= best) continue;
    const long long waves_now = (long long)T * ((units + best * 64 - 1) / (best * 64));
    if (waves_now >= 4096) break;
    if ((units + cands[i] * 64 - 1) / (cands[i] * 64) > 16) break;
    best = cands[i];
  }
  while ((units + best * 64 - 1) / (best * 64) > 16) {  // very wide rows: stay within 16 waves per token
    int next = best;
    for (int i = 0; i < ncand; ++i)
      if (cands[i] > best) {
        next = cands[i];
        break;
      }
    if (next == best) break;
    best = next;
  }
  return best;
}

static int tuned_dispatch_vpl(int H, int T, int forced) {
  static const int c[] = {1, 2, 4, 7, 8, 14, 16};
  for (int v : c)
    if (v == forced) return v;
  // About four waves per token stream best (measured in the full path on 7168- and 4096-wide rows:
  // the command tail of one wave then overlaps the stores of the others); with few tokens the row
  // is split further until there are about 4096 waves (16 per compute unit).
  return split_for(H / 8, T, c, 7);
}

static int tuned_dispatch_fp8_vpl(int H, int T, int forced) {
  static const int c[] = {1, 2, 4};  // more than 4 groups per lane would spill at 128 VGPRs
  for (int v : c)
    if (v == forced) return v;
  return split_for(H / 16, T, c, 3);
}

// One command per row: as many tokens per workgroup as 16 waves hold, and as many workgroups per group as share 64
// pairs (at least 16 groups, so that a handful of tokens does not wait for its slowest).  Where the kernel is bound by its row
// stores a group only keeps its last workgroup busy for longer, and a workgroup pushes its own: above 256 MB of rows, which
// stream to HBM while it runs (dispatch and wait with groups / without, us: 1024 tokens x 20480 86 / 83, 384 x 65536 103 / 98,
// 1536 x 16384 104 / 99; 1536 x 8192 (201 MB) 55 / 66, 512 x 24576 50 / 65; in between it varies: 512 x 40960 82 / 91, 1024 x
// 16384 74 / 69); and above 12288 commands, where whole steps got slower (2048 tokens x 7168 top-8 120 / 117, 4096 tokens 220 /
// 207; 1500 tokens 91 / 92, 1024 tokens 65 / 73), though dispatch and wait by themselves do not (2048 x 7168 60 / 69, 2048 x
// 1024 65 / 63, 16000 x 1024 top-1 53 / 76).  Returns the dynamic LDS bytes of the launch.
static size_t group_cmds_setup(DispatchArgs &a, int waves) {
  a.blocks_per_group = 0;
  if ((a.cmd_mode & EP_CMD_MODE_MASK) != EP_CMD_PER_TOKEN) return 0;
  if (waves < 4 || waves > 16) waves = 16;  // (0 = not set)
  const int tpb = waves / a.parts;
  if (tpb >= 2) a.tokens_per_block = tpb;
  const long long cmds = (long long)a.T * a.K;
  const long long placed = (a.cmd_mode & EP_CMD_NO_PLACEMENT) ? 0 : min(cmds, (long long)a.recv_rows);
  a.blocks_per_group = cmds > kGroupCmdsMax || placed * a.row_bytes > kGroupBytesMax
                           ? 1
                           : max(1, min(64 / a.K, a.T / 16) / a.tokens_per_block);
  return (1 + kLeadWaves) * kSortScratch;
}

// Does a token's row of bf16 leave for the registers together with its pairs?  (See dispatch_bf16_kernel.)  Where all rows are
// few (24 MB) without asking for an expert: such a launch waits for loads more than for memory.  Whole steps, asking / not, us:
// 1500 tokens x 7168 top-6 54.3 / 52.8, 777 x 2944 16.7 / 16.3, 4000 x 2048 57.0 / 56.7; ring off with 19 of 20 tokens dropped,
// 1400 x 7168 5.9 / 6.2, 3000 x 4096 6.3 / 6.2, but 2000 x 7168 6.7 / 8.2.  (FP8 always asks: 1500 x 7168 45.3 / 45.0, 1000 x
// 7168 46.8 / 47.4, and 1400 x 7168 with four of five dropped 6.3 / 6.7.)
static int row_ahead(const DispatchArgs &a) {
  const int cmds = a.cmd_mode & EP_CMD_MODE_MASK;
  if ((cmds != EP_CMD_NONE && cmds != EP_CMD_CHUNK32) || (a.cmd_mode & EP_CMD_NO_PLACEMENT) || a.filter >= 0) return kAheadNone;
  return (long long)a.T * a.H <= 24ll << 19 ? kAheadAll : kAheadNamed;
}

// Ring-on launches take the form with a command wave when it is switched on and the row needs at most 15 data
// waves: returns false when the launch has to take the plain form.
template <int VPL, bool FP8>
static bool launch_pipelined(DispatchArgs a, const Tunables &tune, hipStream_t st, const LaunchTiming *tm) {
  if ((a.cmd_mode & EP_CMD_MODE_MASK) == EP_CMD_NONE || !tune.dispatch_pipeline || a.parts > 15) return false;
  int want = tune.per_token_waves;  // data waves per workgroup, at most
  if (want < 1 || want > 15) want = 12;
  a.tokens_per_block = want / a.parts > 0 ? want / a.parts : 1;
  const int D = a.parts * a.tokens_per_block;
  const int nb = (a.T + a.tokens_per_block - 1) / a.tokens_per_block;
  const int n = a.tokens_per_block * a.K;
  const size_t lds = 16 + (size_t)((n + 1) & ~1) * 2 * sizeof(int2) + kSortScratch;
  // two workgroups per compute unit (256 of them) keep the chip full; each walks its batches with stride gridDim
  const int grid = nb < 1 ? 1 : (nb < 512 ? nb : 512);
  launch_kernel(dispatch_pipelined_kernel<VPL, FP8>, dim3(grid), dim3(64 * (D + 1)), lds, st, tm ? tm->start : nullptr,
                tm ? tm->stop : nullptr, a);
  return true;
}

template <int VPL>
static void launch_dispatch_bf16_t(DispatchArgs a, const Tunables &tune, hipStream_t st, const LaunchTiming *tm) {
  const int nvec = a.H / 8;
  a.parts = (nvec + VPL * 64 - 1) / (VPL * 64);
  if constexpr (VPL != 7 && VPL != 8)  // (they spill there: launch_dispatch asks for 14 and 16 instead)
    if (launch_pipelined<VPL, false>(a, tune, st, tm)) return;
  a.tokens_per_block = a.parts >= 4 ? 1 : 4 / a.parts;
  const size_t lds = group_cmds_setup(a, tune.per_token_waves);
  const int grid = max(1, (a.T + a.tokens_per_block - 1) / a.tokens_per_block);
  auto kernel = a.blocks_per_group ? dispatch_bf16_kernel<VPL, true, kAheadNone> : dispatch_bf16_kernel<VPL, false, kAheadNone>;
  if constexpr (VPL <= 4) {
    if (row_ahead(a) == kAheadAll) kernel = dispatch_bf16_kernel<VPL, false, kAheadAll>;
    if (row_ahead(a) == kAheadNamed) kernel = dispatch_bf16_kernel<VPL, false, kAheadNamed>;
  }
  launch_kernel(kernel, dim3(grid), dim3(64 * a.parts * a.tokens_per_block), lds, st, tm ? tm->start : nullptr,
                tm ? tm->stop : nullptr, a);
}

template <int VPL>
static void launch_dispatch_fp8_t(DispatchArgs a, const Tunables &tune, hipStream_t st, const LaunchTiming *tm) {
  const int npair = a.H / 16;
  a.parts = (npair + VPL * 64 - 1) / (VPL * 64);
  if (launch_pipelined<VPL, true>(a, tune, st, tm)) return;
  a.tokens_per_block = a.parts >= 4 ? 1 : 4 / a.parts;
  const size_t lds = group_cmds_setup(a, tune.per_token_waves);
  const int grid = max(1, (a.T + a.tokens_per_block - 1) / a.tokens_per_block);
  const bool together = a.parts > 1 && min((long long)a.T * a.K, (long long)a.recv_rows) * (a.H + a.H / 32) >= 200000000ll;
  auto kernel = a.blocks_per_group ? dispatch_fp8_kernel<VPL, true, false, false>
                : a.filter >= 0    ? dispatch_fp8_kernel<VPL, false, false, false>
                : together         ? dispatch_fp8_kernel<VPL, false, true, true>
                                   : dispatch_fp8_kernel<VPL, false, true, false>;
  launch_kernel(kernel, dim3(grid), dim3(64 * a.parts * a.tokens_per_block), lds, st, tm ? tm->start : nullptr,
                tm ? tm->stop : nullptr, a);
}

int launch_dispatch(const DispatchArgs &a, int payload, const Tunables &tune, void *stream,
                    const LaunchTiming *timing) {
  hipStream_t st = (hipStream_t)stream;
  // T == 0 with the ring on still launches one (idle) workgroup: it owes the zero-count atomics
  if (a.T <= 0 && (a.cmd_mode & EP_CMD_MODE_MASK) == EP_CMD_NONE) return 0;
  if (payload == EP_BF16) {
    int vpl = tuned_dispatch_vpl(a.H, a.T, tune.dispatch_vpl);
    const int cmds = a.cmd_mode & EP_CMD_MODE_MASK;
    const bool free_choice = !tune.dispatch_vpl && !tune.dispatch_pipeline;
    // One command per row: two 1 KiB slices per wave (rows of up to 8192 channels then still put two tokens
    // into a workgroup, whose first wave pushes for both) beat four by 3-9 us per dispatch, measured for
    // hidden 5120..8192 and 2048..8192 tokens.  The sequenced chunk mode gains 2-6 us from the same shape at
    // 4096 tokens (hidden 5120..8192) and nothing at 8192.
    if (free_choice && (cmds == EP_CMD_PER_TOKEN || cmds == EP_CMD_CHUNK32_ORDERED) &&
        !(a.cmd_mode & EP_CMD_NO_PLACEMENT) && vpl > 2 && (a.H / 8 + 127) / 128 <= 8)
      vpl = 2;
    // Ring off or plain chunk commands: rows that exceed the memory-side cache (256 MB) by a quarter or more have to stream to
    // HBM while the kernel runs; then ONE slice per wave (many small waves, eight 1 KiB stores each) is faster by 5-10 us per
    // 450-900 MB than four slices per wave, which wins below that size by as much when the buffer is the one of the call before
    // - and also where the caller has said that the rows are consumed in place, out of that cache.  Whole steps, four slices /
    // one, into the same buffer and into four in turn, us: 3000 tokens x 7168 top-8 (344 MB) 148.6 / 145.8 and 146.0 / 140.7,
    // 4000 x 5120 (328 MB) 143.9 / 141.8 and 140.7 / 137.8, 2800 x 8192 158.3 / 151.9 and 155.8 / 150.5; 2600 x 7168 (298 MB)
    // 114.0 / 118.3 and 128.2 / 123.9, 2000 x 7168 88.0 / 92.9 and 100.7 / 96.3, 4500 x 4096 (295 MB) 111.8 / 112.2 and 127.5 /
    // 125.9.  The bytes are those of a table without dropped pairs, which only the GPU counts: 3000 x 7168 with a tenth dropped
    // 138.4 / 135.4, three tenths 118.0 / 118.5, half 98.6 / 103.5; 4000 x 5120 133.5 / 130.5, 114.1 / 111.1, 93.6 / 96.4.  A
    // handle with one expert per rank mostly places deduplicated rows, of which a fifth and more are dropped: there from 384 MB
    // on.  Deduplicated steps over 16 groups, 2900 x 7168 221.4 / 228.1, with a tenth dropped 206.2 / 214.9, 3200 x 7168 (367
    // MB) 248.8 / 253.2 and 226.3 / 237.2.  (The sequenced chunk mode, bound by its hottest channel's FIFO, was measured slower
    // with one slice per wave on the skewed workload.)
    const long long rows_at_most = (long long)a.T * a.K < a.recv_rows ? (long long)a.T * a.K : a.recv_rows;
    if (free_choice && !a.cache_hinted && (cmds == EP_CMD_NONE || cmds == EP_CMD_CHUNK32) &&
        rows_at_most * a.H * 2 >= (a.E == a.R ? 384000000ll : 320000000ll) && (a.H / 8 + 63) / 64 <= 16)
      vpl = 1;
    // (7 and 8 vectors per lane make the compiler spill in the form with a command wave: rows that wide take 14 / 16)
    if ((a.cmd_mode & EP_CMD_MODE_MASK) != EP_CMD_NONE && tune.dispatch_pipeline && (vpl == 7 || vpl == 8)) vpl *= 2;
    if ((a.H / 8 + vpl * 64 - 1) / (vpl * 64) > 16) return (int)hipErrorInvalidValue;
    switch (vpl) {
      case 1: launch_dispatch_bf16_t<1>(a, tune, st, timing); break;
      case 2: launch_dispatch_bf16_t<2>(a, tune, st, timing); break;
      case 4: launch_dispatch_bf16_t<4>(a, tune, st, timing); break;
      case 7: launch_dispatch_bf16_t<7>(a, tune, st, timing); break;
      case 8: launch_dispatch_bf16_t<8>(a, tune, st, timing); break;
      case 14: launch_dispatch_bf16_t<14>(a, tune, st, timing); break;
      default: launch_dispatch_bf16_t<16>(a, tune, st, timing); break;
    }
  } else {
    const int vpl = tuned_dispatch_fp8_vpl(a.H, a.T, tune.dispatch_fp8_vpl);
    if ((a.H / 16 + vpl * 64 - 1) / (vpl * 64) > 16) return (int)hipErrorInvalidValue;
    switch (vpl) {
      case 1: launch_dispatch_fp8_t<1>(a, tune, st, timing); break;
      case 2: launch_dispatch_fp8_t<2>(a, tune, st, timing); break;
      default: launch_dispatch_fp8_t<4>(a, tune, st, timing); break;
    }
  }
  return (int)hipGetLastError();
}

}  // namespace ep
