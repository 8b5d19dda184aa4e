// Test double of the HIP runtime calls that libgm's run loop makes, loaded before
// libgm.so (tests/test_error_exits.py) so that the host code runs without a GPU:
// memory is host memory, a launch runs nothing, and the kernel that ends an
// iteration (the one that gets a status slot) is answered with a status that lets
// the loop go on.  It counts the launches that no synchronisation has followed.
#include <cstdint>
#include <cstdlib>
#include <cstring>

namespace {
struct Dim {
  uint32_t x, y, z;
};
struct Slot {  // gm_api.hip StatusSlot: the status block by words, then the number
  int64_t words[64];
};
struct Mirror {
  Slot* slot;
  int64_t seq;
};
int g_launches = 0, g_pending = 0, g_fail_at = 0, g_mallocs = 0, g_events = 0, g_fail_launch = 0;
int g_queries = 0;
int64_t g_iter = 0, g_stop_at = 0;
int g_seq_word = 0;
int g_last = 0;
size_t g_shm = 0;
}  // namespace

extern "C" {
// Malloc number fail_malloc (from 1, since here) and launch number fail_launch fail;
// iteration stop_at ends the run.
void double_reset(int fail_malloc, int fail_launch, int64_t stop_at, int seq_word) {
  g_fail_at = fail_malloc;
  g_fail_launch = fail_launch;
  g_stop_at = stop_at;
  g_seq_word = seq_word;
  g_launches = g_pending = g_mallocs = g_queries = 0;
  g_iter = 0;
}
int double_pending() { return g_pending; }
int double_launches() { return g_launches; }
int double_events() { return g_events; }

int hipMalloc(void** p, size_t n) {
  if (++g_mallocs == g_fail_at) return g_last = 2;  // hipErrorOutOfMemory
  *p = std::calloc(1, n < 64 ? 64 : n);
  return 0;
}
int hipFree(void* p) {
  std::free(p);
  g_pending = 0;  // (waits for the device)
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*) {
  std::memcpy(d, s, n);
  return 0;
}
int hipGetLastError() {
  const int e = g_last;
  g_last = 0;
  return e;
}
const char* hipGetErrorString(int) { return "double"; }
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipStreamSynchronize(void*) {
  g_pending = 0;
  return 0;
}
int hipDeviceSynchronize() {
  g_pending = 0;
  return 0;
}
int hipStreamQuery(void*) {  // hipErrorNotReady, for a while
  return g_pending && ++g_queries < 100 ? 600 : 0;
}
int hipEventCreate(void** e) {
  *e = std::malloc(1);
  ++g_events;
  return 0;
}
int hipEventDestroy(void* e) {
  std::free(e);
  --g_events;
  return 0;
}
int hipEventRecord(void*, void*) { return 0; }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* t, void*, void*) {
  *t = 0.0f;
  return 0;
}
int __hipPushCallConfiguration(Dim, Dim, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* s, void** st) {
  *g = *b = Dim{1, 1, 1};
  *s = g_shm;
  *st = nullptr;
  return 0;
}
// Launch 1 is the initial partition; then the rule, the one-workgroup step and,
// with leaves, their list (sets of at most 32768 regions).
int hipLaunchKernel(const void*, Dim, Dim, void** args, size_t, void*) {
  ++g_launches;
  if (g_launches == g_fail_launch) return g_last = 719;
  ++g_pending;
  const int per = g_stop_at < 0 ? 2 : 3;
  const int64_t stop = g_stop_at < 0 ? -g_stop_at : g_stop_at;
  if (g_iter < stop && g_launches > 1 && (g_launches - 2) % per == 1) {
    const Mirror* m = (const Mirror*)args[6];
    int64_t* w = *(int64_t**)args[0];  // the status block
    ++g_iter;
    w[0] = 20000;            // n_active
    w[1] = 20000;            // n_prev
    w[3] = g_iter;           // iter
    w[4] = g_iter >= stop;   // done
    w[11] = 15000 * g_iter;  // leaf_count
    if (m->slot) {
      std::memcpy(m->slot, w, 8 * g_seq_word);
      ((int64_t*)m->slot)[g_seq_word] = m->seq;
    }
  }
  return 0;
}
}
