// Host driver for the pool of idle workspaces (idle_pool.hpp) on allocation
// functions that count: prints "ok" or the first check that fails.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>

enum hipError_t { hipSuccess, hipErrorUnknown };
static std::map<void*, int> g_freed;
static size_t g_free_bytes = 1 << 20;
static hipError_t hipFree(void* p) {
  ++g_freed[p];
  return hipSuccess;
}
static hipError_t hipMemGetInfo(size_t* fr, size_t* tot) {
  *fr = g_free_bytes;
  *tot = g_free_bytes;
  return hipSuccess;
}
static hipError_t hipGetLastError() { return hipSuccess; }

static bool g_no_host_memory = false;
void* operator new(size_t n) {
  if (g_no_host_memory) throw std::bad_alloc();
  return malloc(n);
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

#include "idle_pool.hpp"

#define CHECK(x)               \
  if (!(x)) {                  \
    printf("line %d: %s\n", __LINE__, #x); \
    return 1;                  \
  }
static void* ptr(int i) { return (void*)(size_t)(4096 * (i + 1)); }

// a buffer serves requests down to eight ninths of it, the smallest that fits first
static int sizes() {
  IdlePool p;
  size_t got = 0;
  CHECK(p.give(ptr(0), 1800) && p.give(ptr(1), 1000) && p.give(ptr(2), 1100));
  CHECK(p.take(900, &got) == ptr(1) && got == 1000);
  CHECK(p.take(1101, &got) == nullptr);
  CHECK(p.take(900, &got) == nullptr);
  CHECK(p.take(1000, &got) == ptr(2) && got == 1100);
  CHECK(p.take(1600, &got) == ptr(0) && got == 1800 && p.bytes() == 0);
  return 0;
}

// at most half of the free memory is kept
static int limits() {
  IdlePool p;
  g_free_bytes = 1000;
  CHECK(!p.give(ptr(0), 501) && p.give(ptr(1), 300) && !p.give(ptr(2), 201) && p.give(ptr(3), 200));
  CHECK(p.bytes() == 500 && g_freed.empty());
  return 0;
}

// every pool's buffers are counted and handed back once
static int all() {
  {
    IdlePool a, b, c;
    b.device = 1;
    CHECK(a.give(ptr(0), 100) && b.give(ptr(1), 200) && c.give(ptr(2), 300));
    CHECK(IdlePool::bytes_on(0) == 400 && IdlePool::bytes_on(1) == 200);
    CHECK(IdlePool::drain_all() && !IdlePool::drain_all());
    CHECK(g_freed.size() == 3 && IdlePool::bytes_on(0) == 0 && IdlePool::bytes_on(1) == 0);
    CHECK(c.give(ptr(3), 100));
  }
  CHECK(g_freed.size() == 4);
  for (auto& f : g_freed) CHECK(f.second == 1);
  return 0;
}

// without host memory for its entry a buffer is refused, and nothing is thrown
// out of the destructor that offers it
static int nohost() {
  IdlePool p;
  g_no_host_memory = true;
  const bool kept = p.give(ptr(0), 100);
  g_no_host_memory = false;
  CHECK(!kept && p.bytes() == 0);
  CHECK(p.give(ptr(0), 100) && p.bytes() == 100);
  return 0;
}

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  const int rc = !strcmp(argv[1], "sizes") ? sizes()
                 : !strcmp(argv[1], "limits") ? limits()
                 : !strcmp(argv[1], "all") ? all()
                 : !strcmp(argv[1], "nohost") ? nohost() : 2;
  if (rc == 0) printf("ok\n");
  return rc;
}
