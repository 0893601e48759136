// Layout (Section 2.1: sizes and destinations are recomputed from the router's output every step): counts,
// exclusive scans and slot indices as an integer counting sort built from LDS bit masks and popcounts.
#include "ep_device.h"

#include <mutex>

namespace ep {

// ------------------------------------------------------------------ layout
// The layout is a counting sort keyed by expert, stable in (source rank, token).
// Tokens are cut into tiles of 64 (one wavefront); f = s * ntiles + tile is the
// "flat" tile index, ascending in exactly the order rows are laid out inside an
// expert.  With hist[f][e] = entries of tile f that chose e,
//   P[f][e]  = sum_{f' < f} hist[f'][e]            (exclusive scan over flat tiles)
//   dst_row  = expert_offset[e] + P[f][e] + rank inside the tile
//   slot     = P[f][e] - P[s * ntiles][e] + rank
//   count[s][e] = P[(s+1) * ntiles][e] - P[s * ntiles][e],  base[s][e] = expert_offset[e] + P[s * ntiles][e].
//
// Kernel 1: one wavefront per tile.  Every lane owns a token and sets its bit in
// a 64-bit LDS mask per expert it chose (a token's experts are distinct, so one
// bit per (token, expert)).  The in-tile stable rank of an entry is the popcount
// of the mask below its lane; the tile histogram is the popcount of the whole
// mask.  The last workgroup to finish (ticket counter, nobody spins) scans the
// histograms (one thread per expert, a batch of flat tiles in registers at a
// time), then the expert totals (one wave scan), and writes every per-expert
// output.  Histograms cross workgroups through device-scope write-through stores
// and cache-bypassing loads, so the hand-over needs no L2 write-back/invalidate
// (measured: a device-scope fence here cost 7 us, mostly flushing other kernels'
// dirty lines).
constexpr int kScanBatch = 32;  // flat tiles a scanning thread holds in registers

__global__ __launch_bounds__(1024) void layout_count_kernel(LayoutArgs a) {
  extern __shared__ unsigned long long s_mask[];  // [waves][E]
  __shared__ int s_off[kMaxExperts + 1];
  __shared__ int s_part[1024];
  __shared__ int s_last;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int W = a.tiles_per_block;  // wavefronts that own a tile; the rest only help with the scan
  const int nblk = max(1, (a.ntiles + W - 1) / W);
  const int s = blockIdx.x / nblk;
  const int tile = wave < W ? (blockIdx.x % nblk) * W + wave : a.ntiles;
  const int E = a.E, K = a.K;
  const int F = a.S * a.ntiles;  // flat tiles

  for (int i = tid; i < W * E; i += blockDim.x) s_mask[i] = 0ull;
  __syncthreads();

  unsigned long long *m = s_mask + (size_t)(wave < W ? wave : 0) * E;
  const int t = tile * kLayoutTile + lane;
  const bool active = tile < a.ntiles && t < a.T;
  const size_t ebase = ((size_t)s * a.T + (active ? t : 0)) * K;
  const unsigned long long below = (1ull << lane) - 1ull;
  if (K <= 8) {  // the token's expert ids stay in registers across the barrier
    int ev[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) ev[k] = (active && k < K) ? a.idx[ebase + k] : -1;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = ev[k];
      bool pend = e >= 0 && e < E;
      if (!pend && e != -1) dev_set_error(a.error, EP_EBOUNDS);
      // Skewed routing sends most lanes of a wave to the same few experts, and an LDS atomic
      // serialises lanes that hit one address.  Peel the two most common values first: their
      // lanes are found with a ballot and one lane writes the whole bit set.
#pragma unroll
      for (int round = 0; round < 2; ++round) {
        const unsigned long long pm = __ballot(pend);
        if (pm == 0) break;
        const int leader = __builtin_ctzll(pm);
        const int e0 = __builtin_amdgcn_readlane(e, leader);
        const unsigned long long same = __ballot(pend && e == e0);
        if (lane == leader) m[e0] |= same;
        pend = pend && e != e0;
      }
      if (pend) atomicOr(&m[e], 1ull << lane);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (active && k < K) a.rank[ebase + k] = (ev[k] >= 0 && ev[k] < E) ? __popcll(m[ev[k]] & below) : -1;
  } else {
    if (active) {
      for (int k = 0; k < K; ++k) {
        const int e = a.idx[ebase + k];
        if (e >= 0 && e < E)
          atomicOr(&m[e], 1ull << lane);
        else if (e != -1)
          dev_set_error(a.error, EP_EBOUNDS);
      }
    }
    __syncthreads();
    if (active) {
      for (int k = 0; k < K; ++k) {
        const int e = a.idx[ebase + k];
        a.rank[ebase + k] = (e >= 0 && e < E) ? __popcll(m[e] & below) : -1;
      }
    }
  }
  if (tile < a.ntiles) {
    int32_t *hist = a.tile_hist + ((size_t)s * a.ntiles + tile) * E;
    for (int e = lane; e < E; e += 64)
      __hip_atomic_store(hist + e, __popcll(m[e]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // ---- last workgroup to arrive does the scans
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // this wave's write-through stores are acknowledged
  __syncthreads();
  if (tid == 0) {
    const unsigned ticket = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = (ticket == gridDim.x - 1);
  }
  __syncthreads();
  if (!s_last) return;
  if (tid == 0) __hip_atomic_store(a.ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // P[*][e]: scan_split threads per expert, each owning a contiguous range of flat tiles
  // (thread = part * E + e, so a wavefront reads consecutive experts of one tile row).
  const int P = a.scan_split;
  const int len = (F + P - 1) / P;
  for (int e_base = 0; e_base < E; e_base += blockDim.x / P) {  // one pass unless E * P > workgroup size
    const int ne = min(E - e_base, (int)blockDim.x / P);
    const bool mine = tid < P * ne;
    const int part = mine ? tid / ne : 0;
    const int e = e_base + (mine ? tid - part * ne : 0);
    const int lo = min(F, part * len), hi = min(F, lo + len);
    int v[kScanBatch];
    int tot = 0;
    if (mine) {
      for (int f0 = lo; f0 < hi; f0 += kScanBatch) {
#pragma unroll
        for (int j = 0; j < kScanBatch; ++j)
          v[j] = (f0 + j < hi) ? __hip_atomic_load(a.tile_hist + (size_t)(f0 + j) * E + e, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT)
                               : 0;
#pragma unroll
        for (int j = 0; j < kScanBatch; ++j) tot += v[j];
      }
      s_part[tid] = tot;
    }
    __syncthreads();
    if (mine) {
      int carry = 0;
      for (int q = 0; q < part; ++q) carry += s_part[q * ne + (e - e_base)];
      for (int f0 = lo; f0 < hi; f0 += kScanBatch) {
        if (hi - lo > kScanBatch) {  // the range did not fit the registers: fetch the batch again
#pragma unroll
          for (int j = 0; j < kScanBatch; ++j)
            v[j] = (f0 + j < hi) ? __hip_atomic_load(a.tile_hist + (size_t)(f0 + j) * E + e, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT)
                                 : 0;
        }
#pragma unroll
        for (int j = 0; j < kScanBatch; ++j) {
          if (f0 + j < hi) a.tile_base[(size_t)(f0 + j) * E + e] = carry;
          carry += v[j];
        }
      }
      if (part == P - 1) {
        a.tile_base[(size_t)F * E + e] = carry;
        a.expert_total[e] = carry;
        s_off[e] = carry;
      }
    }
    __syncthreads();
  }
  __syncthreads();
  if (wave == 0) {  // exclusive scan over experts: 64 lanes x contiguous runs
    const int per = (E + 63) / 64;
    const int lo = min(E, lane * per), hi = min(E, lo + per);
    int sum = 0;
    for (int i = lo; i < hi; ++i) sum += s_off[i];
    const int incl = wave_inclusive_scan(sum, lane);
    int run = incl - sum;
    for (int i = lo; i < hi; ++i) {
      const int v = s_off[i];
      s_off[i] = run;
      a.expert_offset[i] = run;
      run += v;
    }
    if (lane == 63) {
      s_off[E] = incl;
      a.expert_offset[E] = incl;
    }
  }
  __syncthreads();
  for (int i = tid; i < a.S * E; i += blockDim.x) {
    const int ss = i / E, e = i - ss * E;
    const int lo = a.tile_base[(size_t)ss * a.ntiles * E + e], hi = a.tile_base[(size_t)(ss + 1) * a.ntiles * E + e];
    a.count[i] = hi - lo;
    a.base[i] = s_off[e] + lo;
  }
  for (int r = tid; r <= a.R; r += blockDim.x) {
    const int o = s_off[r * a.E_loc];  // r == R reads the end sentinel s_off[E]
    a.rank_offset[r] = o;
    if (r < a.R) a.rank_total[r] = s_off[(r + 1) * a.E_loc] - o;
  }
}

// Kernel 2: per entry, slot and dst_row from the tile prefix and the expert offset.  The entry's own thread reads its id
// and its rank before it writes, so either output may be the table itself (the ranks come in the other one).
__global__ __launch_bounds__(256) void layout_finish_kernel(LayoutArgs a) {
  const long long n = (long long)a.S * a.T * a.K;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int e = a.idx[i];
  if (e < 0 || e >= a.E) {
    a.slot[i] = -1;
    a.dst_row[i] = -1;
    return;
  }
  const long long tk = (long long)a.T * a.K;
  const int s = (int)(i / tk);
  const int t = (int)((i - (long long)s * tk) / a.K);
  const int before = a.tile_base[((size_t)s * a.ntiles + t / kLayoutTile) * a.E + e];
  const int first = a.tile_base[(size_t)s * a.ntiles * a.E + e];
  const int rank = a.rank[i];
  a.slot[i] = before - first + rank;
  a.dst_row[i] = a.expert_offset[e] + before + rank;
}

// ------------------------------------------------- one launch: a workgroup per expert
// Workgroup e reads the WHOLE routing table and needs nothing from any other: the rows of expert e are the entries
// equal to e in table order, and its first row is the number of entries with a smaller id, so a pass that counts
// both gives every output of that expert.  No scratch, no histograms handed from one workgroup to another, no
// second launch - which is what the two kernels above spend their time on, whatever the size of the table.
//
// Each wave owns a run of 256-entry groups, four consecutive entries (a quad) per lane.  A quad that holds e goes
// to the wave's list in LDS (its place and which of the four entries); after one barrier the waves know how many
// entries of e come before theirs and number their lists, 64 quads at a time.
//
// Numbering is two scattered stores per entry, which a compute unit issues at about one address per clock: an expert that
// every token names takes 5 us per 8192 tokens.  With fewer than 256 experts there are compute units to spare, so `parts`
// workgroups count alike for the same expert and each numbers the lists of its own share of the waves (40960 entries of
// one expert 12 us, as one workgroup 30; 65536 of 64 experts, 8192 of them alike, 11 instead of 16).
//
// Bound by instruction issue: every compute unit looks at every entry, about 15 vector instructions per 256 of them on
// pairs of 16-bit ids (32-bit compares and per-lane counts, 35 instructions, took a third longer), the next two groups'
// loads in flight (one: 0.5 us more when the table comes from memory; four, or the whole table: no gain, and longer code,
// which a kernel this short waits for).  On top of that 4 us of launch, first load, barrier and stores.  Measured on MI355X
// against the forms before it, between queued calls (us): 128 entries of 16 experts 4.2 (one-workgroup form with LDS masks
// 5.3), 4096 of 256: 4.1 (11.0), 32768: 7.3 (32-bit compares 8.0, two kernels 16.7), 32768 over 32 sources: 6.8 (7.4, 18.8),
// 65536 of 128 experts 8.3 (9.6), 65536 of 256, Zipf 11.3 (13.1).
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any 4-byte boundary

constexpr int kLayoutAhead = 2;  // groups of a wave whose loads are in flight

__global__ __launch_bounds__(1024) void layout_expert_kernel(LayoutArgs a) {
  extern __shared__ unsigned short s_list[];  // [waves][seg * 64]
  __shared__ int s_cnt[16], s_lt[16], s_rl[16];
  __shared__ int s_first[257];  // entries of e before source s
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int E = a.E, S = a.S, parts = gridDim.y, e = blockIdx.x, part = blockIdx.y;
  const unsigned rank_end = (unsigned)((e / a.E_loc + 1) * a.E_loc);
  const bool first_of_rank = e % a.E_loc == 0;
  const unsigned tk = (unsigned)a.T * a.K, n = (unsigned)S * tk, groups = (n + 255) / 256;
  const unsigned seg = (groups + nw - 1) / nw;                         // groups of one wave
  const unsigned i0 = wave * seg * 256, lim = min(n, i0 + seg * 256);  // its entries
  unsigned short *list = s_list + (size_t)wave * seg * 64;
  if (S > 1)
    for (int s = tid; s <= S; s += blockDim.x) s_first[s] = 0;

  // entries without an expert get -1: the table is shared out over all waves of the grid for that
  const unsigned i_mine = ((part * E + e) * nw + wave) * 64 + lane;
  const int v_mine = i_mine < n ? a.idx[i_mine] : 0;
  int quads = 0;  // list length
  int cnt = 0;    // per lane: entries of e
  // Ids as pairs of 16 bits (saturated: -1 and ids out of range stay above every expert).  min(max(e + 1 - id, 0), 2) is 0,
  // 1 or 2 for an id above, equal to or below e: its bit 0 finds the entries of e, its sum counts the smaller ones.  (A lane
  // sees at most 64 entries.)
  u16x2 weigh = {0, 0}, below = {0, 0};
  const u16x2 e1 = (u16x2)(unsigned short)(e + 1), re = (u16x2)(unsigned short)rank_end;
  auto look = [&](unsigned ib, const i32x4_any &v) {
    const u16x2 p0 = __builtin_amdgcn_cvt_pk_u16(v[0], v[1]), p1 = __builtin_amdgcn_cvt_pk_u16(v[2], v[3]);
    const u16x2 t0 = __builtin_elementwise_min(__builtin_elementwise_sub_sat(e1, p0), (u16x2)(unsigned short)2);
    const u16x2 t1 = __builtin_elementwise_min(__builtin_elementwise_sub_sat(e1, p1), (u16x2)(unsigned short)2);
    weigh += t0;
    weigh += t1;
    const unsigned b0 = __builtin_bit_cast(unsigned, t0), b1 = __builtin_bit_cast(unsigned, t1);
    const bool hit = ((b0 | b1) & 0x10001u) != 0u;
    const unsigned long long any = __builtin_amdgcn_ballot_w64(hit);
    if (any) {
      if (hit) {
        const unsigned u = (b0 & 0x10001u) | (b1 & 0x10001u) << 2, nib = (u | u >> 15) & 15u;
        list[quads + __builtin_amdgcn_mbcnt_hi((unsigned)(any >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)any, 0u))] =
            (unsigned short)((((ib - i0) >> 2) + lane) << 4 | nib);
        cnt += __popc(nib);
      }
      quads += __popcll(any);
    }
    if (first_of_rank) {
      const u16x2 one = (u16x2)(unsigned short)1;
      below += __builtin_elementwise_min(__builtin_elementwise_sub_sat(re, p0), one);
      below += __builtin_elementwise_min(__builtin_elementwise_sub_sat(re, p1), one);
    }
  };
  // full groups first, then what is left of the table (fewer than 256 entries, the last wave's)
  const unsigned nf = n & ~255u, limf = min(lim, nf);
  if (i0 < limf) {
    auto load = [&](unsigned ib) { return *(const i32x4_any *)(a.idx + min(ib, nf - 256u) + lane * 4u); };
    i32x4_any q[kLayoutAhead];
#pragma unroll
    for (int j = 0; j < kLayoutAhead; ++j) q[j] = load(i0 + j * 256u);
#pragma nounroll
    for (unsigned ib = i0; ib < limf; ib += kLayoutAhead * 256u) {
#pragma unroll
      for (int j = 0; j < kLayoutAhead; ++j) {
        const unsigned at = ib + j * 256u;
        if (at >= limf) break;
        const i32x4_any v = q[j];
        q[j] = load(at + kLayoutAhead * 256u);
        look(at, v);
      }
    }
  }
  if (i0 < lim && lim > nf) {
    const unsigned i = nf + lane * 4u;
    i32x4_any v = {-1, -1, -1, -1};
#pragma unroll
    for (unsigned j = 0; j < 4; ++j)
      if (i + j < n) v[j] = a.idx[i + j];
    look(nf, v);
  }
  int lt = ((int)weigh[0] + (int)weigh[1] - cnt) >> 1;  // per lane: entries of an id smaller than e
  int rl = (int)below[0] + (int)below[1];              // ... and (first expert of a rank) below the end of e's rank
  cnt = wave_sum(cnt);
  lt = wave_sum(lt);
  rl = wave_sum(rl);
  if (lane == 0) {
    s_cnt[wave] = cnt;
    s_lt[wave] = lt;
    s_rl[wave] = rl;
  }
  __syncthreads();
  int c_of = 0, lt_of = 0, rl_of = 0;  // lane q: wave q's
  if (lane < nw) {
    c_of = s_cnt[lane];
    lt_of = s_lt[lane];
    rl_of = s_rl[lane];
  }
  const int before = wave_sum(lane < wave ? c_of : 0), total = wave_sum(c_of), off = wave_sum(lt_of),
            end = wave_sum(rl_of);
  if (tid == 0 && part == 0) {
    a.expert_total[e] = total;
    a.expert_offset[e] = off;
    if (e == E - 1) a.expert_offset[E] = a.rank_offset[a.R] = off + total;
    if (first_of_rank) {
      a.rank_offset[e / a.E_loc] = off;
      a.rank_total[e / a.E_loc] = end - off;
    }
  }
  if (S > 1) {  // entries of e per source, then their prefix
    for (int p0 = 0; p0 < quads; p0 += 64) {
      const int p = p0 + lane;
      const unsigned q = p < quads ? list[p] : 0u;
      unsigned nib = q & 15u;
      if (p0 + 64 <= quads) {  // 64 quads, most often of one source: one addition
        const unsigned lo = (i0 + (list[p0] >> 4) * 4u) / tk, hi = (i0 + (list[p0 + 63] >> 4) * 4u + 3u) / tk;
        if (lo == hi) {
          const int c = wave_sum(__popc(nib));
          if (lane == 0) atomicAdd(&s_first[lo + 1], c);
          continue;
        }
      }
      for (; nib; nib &= nib - 1) atomicAdd(&s_first[(i0 + (q >> 4) * 4 + __builtin_ctz(nib)) / tk + 1], 1);
    }
    __syncthreads();
    if (wave == 0) {
      int carry = 0;
      for (int s0 = 0; s0 < S; s0 += 64) {
        const int s = s0 + lane, c = s < S ? s_first[s + 1] : 0;
        const int incl = carry + wave_inclusive_scan(c, lane);
        if (s < S) {
          s_first[s + 1] = incl;
          if (part == 0) {
            a.count[(size_t)s * E + e] = c;
            a.base[(size_t)s * E + e] = off + incl - c;
          }
        }
        carry = __builtin_amdgcn_readlane(incl, 63);
      }
    }
    __syncthreads();
  } else if (tid == 0 && part == 0) {
    a.count[e] = total;
    a.base[e] = off;
  }
  // the r-th entry of e in table order gets row off + r
  int run = before;
  if (parts > 1 && wave % parts != part) quads = 0;  // (another workgroup of this expert numbers these)
  for (int p0 = 0; p0 < quads; p0 += 64) {
    const int p = p0 + lane;
    const unsigned q = p < quads ? list[p] : 0u;
    unsigned nib = q & 15u;
    const int c = __popc(nib);
    int r = run;
    if (__ballot(c > 1) == 0) {  // (always so when 4 divides K: a token's experts are distinct)
      r += lane;
      run += min(64, quads - p0);
    } else {
      const int incl = wave_inclusive_scan(c, lane);
      r += incl - c;
      run += __builtin_amdgcn_readlane(incl, 63);
    }
    for (; nib; nib &= nib - 1, ++r) {
      const unsigned i = i0 + (q >> 4) * 4 + __builtin_ctz(nib);
      a.slot[i] = r - (S > 1 ? s_first[i / tk] : 0);
      a.dst_row[i] = off + r;
    }
  }
  for (unsigned i = i_mine; i < n; i += parts * E * nw * 64) {
    const int w = i == i_mine ? v_mine : a.idx[i];
    if (w >= 0 && w < E) continue;
    if (w != -1) dev_set_error(a.error, EP_EBOUNDS);
    a.slot[i] = a.dst_row[i] = -1;
  }
}

// ------------------------------------------------- scratch that nobody allocates
// For callers that cannot allocate (ep_layout_static): the tile histograms, the tile prefixes, the ticket
// and an error sink live in a file-scope device array.  Every GPU holds its own copy at its own address
// until the process ends, so the address is looked up once per device, with that device current, and
// host code only ever uses the looked-up pointer (the array's name is a host-side stand-in, not a
// device address).
struct StaticLayoutScratch {
  unsigned ticket[64];  // one word used; a 256-byte line of its own
  int error_sink[64];   // where device-side errors go when the caller passes no status word
  int32_t hist[kStaticLayoutEntries];
  int32_t base[kStaticLayoutEntries];
};
static __device__ __align__(256) unsigned char scratch[sizeof(StaticLayoutScratch)];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kMaxDevices] = {};

int static_layout_scratch(LayoutArgs *a) {
  int dev = -1;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return (int)err;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  void *p = nullptr;
  {
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (err != hipSuccess) return (int)err;
      if (!p) return (int)hipErrorInvalidSymbol;
      g_scratch_ptr[dev] = p;
    }
    p = g_scratch_ptr[dev];
  }
  if (a) {
    StaticLayoutScratch *sc = (StaticLayoutScratch *)p;
    a->ticket = sc->ticket;
    a->tile_hist = sc->hist;
    a->tile_base = sc->base;
    if (!a->error) a->error = sc->error_sink;
  }
  return 0;
}

int launch_layout(const LayoutArgs &a, const Tunables &tune, void *stream, const LaunchTiming *timing) {
  hipStream_t st = (hipStream_t)stream;
  if (layout_takes_one_launch(a, tune)) {
    const int groups = (int)(((long long)a.S * a.T * a.K + 255) / 256);
    const int waves = groups < 1 ? 1 : (groups > 16 ? 16 : groups);
    const size_t lds = (size_t)waves * ((groups + waves - 1) / waves) * 64 * sizeof(unsigned short);
    // workgroups of an expert (up to 2048 tokens one numbers its entries in a microsecond)
    const int parts = (long long)a.S * a.T <= 2048 ? 1 : max(1, min(waves, 256 / a.E));
    launch_kernel(layout_expert_kernel, dim3(a.E, parts), dim3(64 * waves), lds, st, timing ? timing->start : nullptr,
                  timing ? timing->stop : nullptr, a);
    return (int)hipGetLastError();
  }
  // Workgroups are 1024 threads so that the last one has many hands for the scan, but only a few
  // wavefronts of each own a tile: the LDS atomics of one tile then compete with few others.
  const int kBlock = 1024;
  int W = tune.layout_tpb;
  if (W != 1 && W != 2 && W != 4 && W != 8 && W != 16) W = 4;
  while (W > 1 && (size_t)W * a.E * sizeof(unsigned long long) > 65536 - 12288) W >>= 1;
  LayoutArgs b = a;
  b.rank = a.slot != a.idx ? a.slot : a.dst_row;
  b.tiles_per_block = W;
  b.scan_split = 1;  // threads per expert in the scan: a power of two, at most 16, all in one workgroup
  while (b.scan_split < 16 && b.scan_split * 2 * a.E <= kBlock) b.scan_split *= 2;
  const int nblk = (a.ntiles + W - 1) / W;
  const int grid1 = a.S * (nblk > 0 ? nblk : 1);
  const size_t lds = (size_t)W * a.E * sizeof(unsigned long long);
  const long long n = (long long)a.S * a.T * a.K;  // entries the second kernel finishes
  launch_kernel(layout_count_kernel, dim3(grid1), dim3(kBlock), lds, st, timing ? timing->start : nullptr,
                timing && n <= 0 ? timing->stop : nullptr, b);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return (int)err;
  if (n > 0) {
    launch_kernel(layout_finish_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, nullptr,
                  timing ? timing->stop : nullptr, b);
    err = hipGetLastError();
  }
  return (int)err;
}

}  // namespace ep
