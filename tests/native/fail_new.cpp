// Preloaded in front of libstdc++: host allocations of at least `limit` bytes fail while limit > 0.
#include <atomic>
#include <cstdlib>
#include <new>

static std::atomic<std::size_t> limit{0};
extern "C" void fail_new_at(std::size_t bytes) { limit = bytes; }

void *operator new(std::size_t n) {
  const std::size_t l = limit;
  if (l > 0 && n >= l) throw std::bad_alloc();
  if (void *p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
