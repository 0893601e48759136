// Stand-alone driver for the copies of the proxy threads on their way through the shared batches, built with sanitizers by
// tests/test_host_copy_pool.py.  A "device" thread copies the batches in order and marks their events late; the Writes
// come from producer threads over all channels, in bursts and in trickles, into heaps that change between rounds, and once
// while batches of the old heaps are under way and open.
#include <condition_variable>
#include <cstdio>

#include "../../paper_2512_19849_amd/csrc/ep_host.h"
using namespace ep;

struct Job {
  const CopyDesc *d;  // (read when the batch is copied, as the kernel for many rows does)
  int n;
  const char *src;
  char *dst;
  std::atomic<int> *pending;
};
static std::mutex jobs_mu;
static std::condition_variable jobs_cv;
static std::deque<Job> jobs;
static bool quit = false;
static std::atomic<bool> hold{false};  // the device copies nothing

static void device() {
  for (int n = 0;; ++n) {
    std::unique_lock<std::mutex> l(jobs_mu);
    jobs_cv.wait(l, [] { return quit || !jobs.empty(); });
    if (jobs.empty()) return;
    Job j = std::move(jobs.front());
    jobs.pop_front();
    l.unlock();
    while (hold.load()) std::this_thread::yield();
    for (const CopyDesc *d = j.d; d < j.d + j.n; ++d) memcpy(j.dst + d->dst16 * 16ull, j.src + d->src16 * 16ull, d->len16 * 16ull);
    std::this_thread::sleep_for(std::chrono::microseconds(n % 5 * 20));
    j.pending->store(0, std::memory_order_release);
  }
}
extern "C" hipError_t hipEventQuery(hipEvent_t e) {
  return ((std::atomic<int> *)e)->load(std::memory_order_acquire) ? hipErrorNotReady : hipSuccess;
}
namespace ep {
int launch_layout(const LayoutArgs &, const Tunables &, void *, const LaunchTiming *) { return 0; }
int launch_dispatch(const DispatchArgs &, int, const Tunables &, void *, const LaunchTiming *) { return 0; }
int launch_combine(const CombineArgs &, const Tunables &, void *, const LaunchTiming *) { return 0; }
int launch_fill_u32(uint32_t *, uint32_t, long long, void *) { return 0; }
int launch_fp8_unpack(const void *, long long, int, unsigned, void *, float *, void *) { return 0; }
int static_layout_scratch(LayoutArgs *) { return 0; }
int launch_recv_wait(const RecvWaitArgs &, void *) { return 0; }
int launch_barrier(const RingDev &, void *) { return 0; }
int launch_dedup(const DedupArgs &, void *) { return 0; }
int launch_gather_index(const GatherIndexArgs &, void *) { return 0; }
int launch_combine_partial(const CombinePartialArgs &, void *) { return 0; }
int launch_bw_probe(int, const void *, void *, long long, void *) { return 0; }
int launch_row_probe(int, const int32_t *, int, long long, int, long long, void *, void *, void *) { return 0; }
int launch_ht_ring(const HtRingArgs &, const Tunables &, void *) { return 0; }
int launch_fifo_stress(const RingDev &, int, int, unsigned long long *, unsigned long long *, void *) { return 0; }
int launch_copy_batch(const CopyBatchArgs &b, void *) {
  Job j{b.host_descs, b.n, b.src_base, b.dst_base, (std::atomic<int> *)b.done};
  unsigned most = 0, least = ~0u;
  for (int i = 0; i < b.n; ++i) most = std::max(most, j.d[i].len16), least = std::min(least, j.d[i].len16);
  if (b.n < 1 || b.n > kCopyBatchMax || most != b.max_len16 || least != b.min_len16 || j.pending->exchange(1)) return 1;
  std::lock_guard<std::mutex> l(jobs_mu);
  jobs.push_back(std::move(j));
  jobs_cv.notify_one();
  return 0;
}
}  // namespace ep

// Heaps change with as many batches of the old ones under way as may be, and copies of the old ones in the open batch.
static int change_under_way(ep_handle *h, char *a, char *b, size_t bytes) {
  CopyPool &C = h->copies;
  const auto until = [](auto f) {
    while (!f()) std::this_thread::yield();
  };
  const auto heaps = [&](int i) {
    h->src_base.store(a + i * bytes);
    h->dst_base.store(b + i * bytes);
  };
  const auto write = [&](int e, uint32_t from, uint32_t row) {
    uint64_t idx;
    ep_host_push(h, e, 1u << 28 | (uint32_t)e, 16, from * 16, row * 16, &idx);
    return idx;
  };
  memset(b, 0, 2 * bytes);
  heaps(0);
  hold.store(true);
  const uint64_t before = C.launched.load();
  uint32_t n = 0;
  for (int i = 0; i < CopyPool::kAhead; ++i) {
    write(0, n * 7, n), ++n;
    until([&] { return C.launched.load() == before + i + 1; });
  }
  write(0, n * 7, n), ++n;
  until([&] {
    std::lock_guard<std::mutex> l(C.mu);
    return C.open.n == 1;
  });
  heaps(1);
  for (int e = 0; e < 4; ++e) {  // (a channel, and with it a proxy thread, for each)
    const uint64_t idx = write(e, 1000 + e, 100 + e);
    until([&] { return ep_host_check_completion(h, e, idx) == 1; });
  }
  std::this_thread::sleep_for(std::chrono::milliseconds(5));  // (they meet the open batch)
  int bad = 0;
  {
    std::lock_guard<std::mutex> l(C.mu);
    bad += C.open.n != 1 || C.open.dst_base != b || C.launched.load() != before + CopyPool::kAhead;
  }
  hold.store(false);
  ep_host_expect_atomics(h, 4);
  for (uint32_t e = 0; e < 4; ++e) {
    uint64_t idx;
    ep_host_push(h, (int)e, 2u << 28 | e, e ? 1 : 1 + n, 0, e, &idx);
  }
  bad += ep_wait(h) != 0;
  for (uint32_t r = 0; r < n; ++r) bad += memcmp(b + r * 256, a + r * 7 * 256, 256) != 0;
  for (uint32_t e = 0; e < 4; ++e) bad += memcmp(b + bytes + (100 + e) * 256, a + bytes + (1000 + e) * 256, 256) != 0;
  for (size_t i = 0; i < 256; ++i) bad += b[100 * 256 + i] != 0 || b[bytes + i] != 0;
  return bad;
}

// The proxy keeps polling while nothing is copied: one thread's commands, more than the batches and the ring hold.
static int backlog(ep_handle *h, char *a, char *b, size_t bytes) {
  const uint32_t per = 9000, rows = (uint32_t)(bytes / 256);
  memset(b, 0, bytes);
  h->src_base.store(a);
  h->dst_base.store(b);
  hold.store(true);
  ep_host_expect_atomics(h, 4);
  int bad = 0;
  uint64_t idx = 0;
  for (uint32_t i = 0; i < 4 * per && !bad; ++i)
    bad += ep_host_push(h, 0, 1u << 28 | i % 4, 16, i * 7 % rows * 16, i % rows * 16, &idx) != 0;
  for (uint32_t e = 0; e < 4; ++e) bad += ep_host_push(h, 0, 2u << 28 | e, per, 0, e, &idx) != 0;
  for (int i = 0; i < 2000 && !ep_host_check_completion(h, 0, idx); ++i) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  bad += ep_host_check_completion(h, 0, idx) != 1 || h->copies.number - h->copies.done.load() > CopyPool::kAhead;
  hold.store(false);
  bad += ep_wait(h) != 0;
  for (uint32_t i = 4 * per - rows; i < 4 * per; ++i) bad += memcmp(b + i % rows * 256, a + i * 7 % rows * 256, 256) != 0;
  return bad;
}

int main() {
  std::thread dev(device);
  ep_config c{};
  c.num_ranks = 4, c.num_experts = 16, c.top_k = 2, c.hidden = 128, c.max_tokens = 65536, c.num_src = 1, c.num_channels = 8;
  c.ring_entries = 8192, c.num_proxy_threads = 4, c.spin_timeout_ms = 20000, c.flags = EP_FLAG_HOST_ONLY;
  ep_handle *h = nullptr;
  if (ep_proxy_start(&c, &h)) return 1;
  std::atomic<int> events[CopyPool::kSlots] = {};
  for (int i = 0; i < CopyPool::kSlots; ++i) h->copies.events[i] = (hipEvent_t)&events[i];
  std::vector<CopyDesc> descs((size_t)CopyPool::kSlots * kCopyBatchMax);
  h->copies.descs = descs.data();
  const size_t rows = 16 * 2000, bytes = rows * 256;
  std::vector<char> a(bytes * 2), b(bytes * 2);
  for (size_t i = 0; i < a.size(); ++i) a[i] = (char)(i * 2654435761u >> 13);
  h->src_bytes = h->dst_bytes = bytes;
  int bad = 0;
  for (int rep = 0; rep < 6; ++rep) {
    const char *src = a.data() + rep % 3 / 2 * bytes;
    char *dst = b.data() + rep % 2 * bytes;
    memset(dst, 0, bytes);
    h->src_base.store(src);
    h->dst_base.store(dst);
    const int per = rep < 2 ? 2000 : rep == 2 ? 1 : 40 * rep;  // Writes of an expert: of one row, every third of half a row
    ep_host_expect_atomics(h, 16);
    std::vector<std::thread> ts;
    for (int p = 0; p < 8; ++p)
      ts.emplace_back([&, p] {
        for (int e = p; e < 16; e += 8) {
          const uint32_t to = (uint32_t)(e / 4) << 12 | (uint32_t)(e % 4);
          uint64_t idx;
          for (int i = 0; i < per; ++i) {
            const size_t r = (size_t)e * per + i;
            ep_host_push(h, e % 8, 1u << 28 | to, i % 3 ? 16 : 8, (uint32_t)(r * 7 % rows * 16), (uint32_t)(r * 16), &idx);
            if (rep > 2 && i % 16 == 0) std::this_thread::sleep_for(std::chrono::microseconds(30));
          }
          ep_host_push(h, e % 8, 2u << 28 | to, per, 0, e % 4, &idx);
        }
      });
    for (auto &t : ts) t.join();
    bad += ep_wait(h) != 0;
    for (size_t r = 0; r < 16ull * per; ++r) bad += memcmp(dst + r * 256, src + r * 7 % rows * 256, r % per % 3 ? 256 : 128) != 0;
  }
  bad += change_under_way(h, a.data(), b.data(), bytes);
  bad += backlog(h, a.data(), b.data(), bytes);
  h->copies.descs = nullptr;
  for (auto &e : h->copies.events) e = nullptr;
  ep_proxy_stop(h);
  std::unique_lock<std::mutex> l(jobs_mu);
  quit = true;
  l.unlock();
  jobs_cv.notify_one();
  dev.join();
  printf("bad %d\n", bad);
  return bad != 0;
}
