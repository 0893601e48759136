// The wait for room of a Push (ring_publish_run, included by the test from ep_device.h as it stands there) by one lane
// on the CPU: a clock that only the kernel's sleep advances, and a proxy that pops at given times.
#include <cstdint>
#include <cstdio>

#define EP_DEV static
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0
enum { EP_ETIMEOUT = -5, kHeadStride = 1 };

struct u32x4 {
  unsigned w[4];
};
struct RingDev {
  unsigned long long *head, *cached_head, *stalls;
  int *error;
  unsigned *refresh_lock;
  unsigned entries;
  unsigned long long timeout_ticks;
};

static unsigned long long now, pops[2], head, cached_head, stalls, stored;
static int error;

static unsigned long long wall_clock64() { return now; }
static void __builtin_amdgcn_s_sleep(int) {
  ++now;
  head = (now >= pops[0]) + (now >= pops[1]);
}
static unsigned long long __ballot(bool b) { return b; }
static void dev_set_error(int *e, int code) { *e = code; }
template <class T>
static T exchange(T *p, T v) {
  const T old = *p;
  *p = v;
  return old;
}
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
#define __hip_atomic_exchange(p, v, order, scope) exchange(p, v)
#define __hip_atomic_fetch_add(p, v, order, scope) (*(p) += (v))
#define __hip_atomic_fetch_max(p, v, order, scope) (*(p) = *(p) > (v) ? *(p) : (v))
static unsigned long long ring_head(const RingDev &r, unsigned) { return *r.cached_head; }
static void ring_store(const RingDev &, unsigned, unsigned long long, const u32x4 &) { ++stored; }

#include RING_PUBLISH_RUN

// Ring of two slots, both taken; the pair has Idx 2 and 3 and the proxy pops 0 and 1 at the given times; limit 100.
static void pair(unsigned long long first, unsigned long long second) {
  unsigned lock = 0;
  now = head = cached_head = stalls = stored = 0;
  error = 0;
  pops[0] = first, pops[1] = second;
  const RingDev r{&head, &cached_head, &stalls, &error, &lock, 2, 100};
  const unsigned long long idx = ring_publish_run<2>(r, 0, 2, 0, u32x4{}, u32x4{});
  printf("%lld error %d stored %llu stalls %llu\n", (long long)idx, error, stored, stalls);
}

int main() {
  pair(10, 10);
  pair(60, 120);
  pair(60, 1000);
  pair(1000, 2000);
}
