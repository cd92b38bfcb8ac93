// host_copy.cpp -- field arrays between the device and pageable host memory.
//
// A copy into a caller's ordinary memory goes through the runtime's pinned
// buffer on one thread, and the destination of a read-back is usually fresh
// memory, so that thread also takes a page fault every 4 KiB: 268 MB (c, u
// and p of 2048^2, N = 5) took 30 ms where the link needs 5.  Large copies
// here are cut into chunks that several threads move: each takes the next
// chunk, has it copied into a pinned buffer of its own and copies it on (14
// ms).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

#include "host_internal.h"

namespace nplbm {

namespace {

constexpr size_t kChunk = (size_t)1 << 20;  // bytes of one chunk
// Copies below this go the plain way.  The copy itself gains from 32 MB on, but
// a caller with as many threads of its own as there are cores now and then
// finds one of them pushed aside after it, and waits up to 20 ms at its own
// barrier: any other threads of the process disturb the wake-up of those, also
// threads that make no runtime call, and it happens (in one pass of a hundred)
// without them.  The line is where copy and what follows cross: get_c of one
// array and its conversion by 16 OpenMP threads on 16 cores, mean of 100
// passes, plain / threads: 24 MB 1.8 - 2.7 / 3.9 - 4.2 ms, 32 MB 4.0 / 4.4 -
// 4.7, 48 MB 6.0 / 6.3 - 7.0, 64 MB 8.8 - 9.3 / 8.2 - 8.4, 96 MB 14.2 - 14.9 /
// 11.3 - 12.0.  A frame of 168 + 67 + 34 MB: 35.1 - 35.9 ms / 21.8 - 24.2, the
// worst of 150 passes 55 - 58 / 44 - 47.
constexpr size_t kLarge = 56 * kChunk;
constexpr int kMaxThreads = 8;

// The pinned buffers, shared by every domain and server of the process: at
// most kMaxBuffers, allocated as they are first needed and freed when the
// last domain and server is gone.  A copy takes what is free for its
// duration and goes the plain way where nothing is.
constexpr int kMaxBuffers = 2 * kMaxThreads;
std::mutex g_mu;
std::vector<void *> g_free;
int g_made = 0, g_users = 0;

void free_buffer(void *p) {
  if (hipHostFree(p) != hipSuccess) forget_hip_error();
  --g_made;
}

int take_buffers(void **buf, int want) {
  std::lock_guard<std::mutex> lk(g_mu);
  int n = 0;
  while (n < want && !g_free.empty()) {
    buf[n++] = g_free.back();
    g_free.pop_back();
  }
  while (n < want && g_made < kMaxBuffers) {
    void *p = nullptr;
    if (hipHostMalloc(&p, kChunk, hipHostMallocPortable) != hipSuccess) {
      forget_hip_error();  // fewer buffers, or none, will do
      break;
    }
    ++g_made;
    buf[n++] = p;
  }
  return n;
}

void give_buffers(void **buf, int n) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (int i = 0; i < n; ++i)
    if (g_users > 0)
      g_free.push_back(buf[i]);
    else
      free_buffer(buf[i]);
}

// f(thread number) on up to n threads, the caller's among them; fewer where
// the system gives no more.
template <typename F>
void on_threads(int n, F f) {
  std::vector<std::thread> th;
  try {
    for (int i = 1; i < n; ++i) th.emplace_back(f, i);
  } catch (const std::system_error &) {
  } catch (const std::bad_alloc &) {
  }
  f(0);
  for (auto &t : th) t.join();
}

int thread_count(size_t pieces) {
  const unsigned hw = std::thread::hardware_concurrency();
  return (int)std::min<size_t>({(size_t)kMaxThreads, (size_t)std::max(1u, hw), pieces});
}

}  // namespace

void copy_users(int change) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_users += change;
  if (g_users > 0) return;
  for (void *p : g_free) free_buffer(p);
  g_free.clear();
}

hipError_t copy_to_host(void *dst, const void *src, size_t bytes, hipStream_t st) {
  void *buf[kMaxThreads];
  const size_t pieces = (bytes + kChunk - 1) / kChunk;
  int nb = 0, dev = 0;
  if (bytes >= kLarge && hipGetDevice(&dev) == hipSuccess)
    nb = take_buffers(buf, thread_count(pieces));
  if (nb == 0) {
    hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
    return e == hipSuccess ? hipStreamSynchronize(st) : e;
  }
  std::atomic<size_t> next{0};
  std::atomic<int> err{(int)hipSuccess};
  on_threads(nb, [&](int t) {
    hipEvent_t ev = nullptr;
    hipError_t e = hipSetDevice(dev);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    while (e == hipSuccess && err.load() == (int)hipSuccess) {
      const size_t i = next.fetch_add(1);
      if (i >= pieces) break;
      const size_t off = i * kChunk, n = std::min(kChunk, bytes - off);
      e = hipMemcpyAsync(buf[t], static_cast<const char *>(src) + off, n, hipMemcpyDeviceToHost,
                         st);
      if (e == hipSuccess) e = hipEventRecord(ev, st);
      if (e == hipSuccess) e = hipEventSynchronize(ev);
      if (e == hipSuccess) std::memcpy(static_cast<char *>(dst) + off, buf[t], n);
    }
    if (e != hipSuccess) err.store((int)e);
    if (ev) (void)hipEventDestroy(ev);
  });
  // after an error copies into the buffers may still be in flight
  hipError_t e = (hipError_t)err.load();
  if (e != hipSuccess) (void)hipStreamSynchronize(st);
  give_buffers(buf, nb);
  return e;
}

// First node whose c_k do not sum to 1 (within 1e-9; a c that is not finite
// makes the sum not finite), or n.  Blocks of nodes, phase by phase, so that
// every array is read in order.
size_t first_bad_sum(const double *c, int N, size_t n) {
  constexpr size_t kBlock = 2048;
  const size_t blocks = (n + kBlock - 1) / kBlock;
  std::atomic<size_t> next{0}, bad{n};
  auto scan = [&](int) {
    double s[kBlock];
    for (size_t b; (b = next.fetch_add(1)) < blocks;) {
      const size_t a = b * kBlock, m = std::min(kBlock, n - a);
      if (a >= bad.load()) return;  // a lower block holds one already
      std::fill(s, s + m, 0.0);
      for (int k = 0; k < N; ++k) {
        const double *ck = c + (size_t)k * n + a;
        for (size_t j = 0; j < m; ++j) s[j] += ck[j];
      }
      size_t wrong = 0;
      for (size_t j = 0; j < m; ++j) wrong += !(std::fabs(s[j] - 1.0) <= 1e-9);
      if (!wrong) continue;
      size_t j = 0;
      while (std::fabs(s[j] - 1.0) <= 1e-9) ++j;
      size_t was = bad.load();
      while (a + j < was && !bad.compare_exchange_weak(was, a + j)) {
      }
      return;
    }
  };
  if (n * N < ((size_t)1 << 22))
    scan(0);
  else
    on_threads(thread_count(blocks), scan);
  return bad.load();
}

bool all_finite(const double *v, size_t n) {
  double z[8] = {0.0};  // v * 0 is 0, or NaN where v is not finite
  size_t i = 0;
  for (; i + 8 <= n; i += 8)
    for (int j = 0; j < 8; ++j) z[j] += v[i + j] * 0.0;
  for (; i < n; ++i) z[0] += v[i] * 0.0;
  return z[0] + z[1] + z[2] + z[3] + z[4] + z[5] + z[6] + z[7] == 0.0;
}

}  // namespace nplbm
