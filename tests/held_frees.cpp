// Order of waits and releases of a context (mgd::Ctx), without a GPU: this
// program's hipStreamSynchronize takes the runtime's place, and the context's
// allocator records every release.  Exits 0 when each held-back buffer is
// released only after a wait that began once the buffer had been let go, and an
// allocation that fails first releases what is held back.
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>

#include "common.hpp"

static std::map<void*, int> g_freed;     // buffer -> times released
static std::function<void()> g_in_wait;  // what another thread does meanwhile
static size_t g_room = size_t(1) << 40;   // bytes left to the allocator
static std::map<void*, size_t> g_size;
static hipError_t g_result = hipSuccess;

extern "C" hipError_t hipStreamSynchronize(hipStream_t) {
  if (g_in_wait) g_in_wait();
  return g_result;
}

static int g_bad = 0;
static void expect(bool ok, const char* what) {
  if (!ok) {
    std::printf("failed: %s\n", what);
    ++g_bad;
  }
}

int main() {
  mgd::Ctx c;
  c.has_alloc = true;
  c.alloc.alloc = [](size_t n, void*, void*) -> void* {
    if (n > g_room) return nullptr;
    g_room -= n;
    void* p = std::malloc(n);
    g_size[p] = n;
    return p;
  };
  c.alloc.free = [](void* p, void*, void*) {  // kept, so that no address comes twice
    g_room += g_size[p];
    ++g_freed[p];
  };
  const size_t n = size_t(1) << 20;  // not from a chunk
  {
    mgd::DeferFrees frees(&c);
    void* before = c.dmalloc(n);
    void* meanwhile = c.dmalloc(n);
    c.dfree(before);
    // the setup's thread launches a kernel on `meanwhile` and lets it go while a
    // thread that closes a handle waits
    g_in_wait = [&] { c.dfree(meanwhile); };
    c.sync();
    g_in_wait = nullptr;
    expect(g_freed[before] == 1, "a buffer let go before the wait is released after it");
    expect(g_freed[meanwhile] == 0, "a buffer let go during the wait outlives it");
    c.sync();
    expect(g_freed[meanwhile] == 1, "the next wait releases it");

    // a wait that fails releases nothing
    void* kept = c.dmalloc(n);
    c.dfree(kept);
    g_result = hipErrorUnknown;
    bool threw = false;
    try {
      c.sync();
    } catch (const std::exception&) {
      threw = true;
    }
    g_result = hipSuccess;
    expect(threw, "a failed wait is reported");
    expect(g_freed[kept] == 0, "a failed wait releases nothing");
    c.sync();
    expect(g_freed[kept] == 1, "a later wait does");
  }
  {
    void* a = c.dmalloc(n);
    int released_in_wait = -1;
    {
      mgd::DeferFrees outer(&c);
      {
        mgd::DeferFrees inner(&c);
        c.dfree(a);
      }
      expect(g_freed[a] == 0, "an inner scope holds on");
      g_in_wait = [&] { released_in_wait = g_freed[a]; };
    }
    g_in_wait = nullptr;
    expect(released_in_wait == 0, "the end of a scope waits first");
    expect(g_freed[a] == 1, "the end of a scope releases what is left");
  }
  {
    // memory for three buffers: what is held back makes room, small or large
    for (size_t size : {n, size_t(4096)}) {
      g_room = 3 * n;
      mgd::DeferFrees frees(&c);
      bool got = true;
      try {
        for (int k = 0; k < 3 * (int)(n / size) + 2; ++k) c.dfree(c.dmalloc(size));
      } catch (const std::exception&) {
        got = false;
      }
      expect(got, "an allocation that fails releases what is held back and tries again");
      bool refused = false;
      try {
        (void)c.dmalloc(4 * n);
      } catch (const std::exception&) {
        refused = true;
      }
      expect(refused, "more than there is stays refused");
    }
  }
  if (!g_bad) std::printf("ok\n");
  return g_bad ? 1 : 0;
}
