// CPU harness of the policy that keeps device blocks between calls
// (mcrt_blocks.hpp): one store, blocks named by number, events that the test
// ends.  Counts the allocations the policy makes.
#include <cstdlib>
#include <new>

#include "mcrt_blocks.hpp"

using namespace mcrt;

namespace {
unsigned long long g_news = 0;
BlockStore* g_store = nullptr;
bool g_over[4096];  // by block number: its last use has ended

constexpr size_t kPerThread = 2;  // the stream that every thread has of its own
const void* stream(int s) {
  return stream_key(reinterpret_cast<const void*>((size_t)s), reinterpret_cast<const void*>(kPerThread));
}
int number(const Block& b) { return (int)reinterpret_cast<size_t>(b.ptr); }
bool over(const Block& b) { return g_over[number(b)]; }
}  // namespace

void* operator new(size_t n) {
  ++g_news;
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {

void blocks_reset(void) {
  delete g_store;
  g_store = new BlockStore;
  for (bool& o : g_over) o = true;
  g_news = 0;
}
unsigned long long blocks_news(void) { return g_news; }
void blocks_call(void) { g_store->call(); }
void blocks_set_over(int id, int over) { g_over[id] = over != 0; }
int blocks_keep(int id, unsigned long long bytes, int dev, int st) {
  Block b{};
  b.ptr = reinterpret_cast<unsigned char*>((size_t)id);
  b.bytes = bytes;
  b.dev = dev;
  b.st = stream(st);
  return g_store->keep(b);
}
int blocks_take(unsigned long long bytes, int dev, int st) {
  Block b;
  return g_store->take(bytes, dev, stream(st), over, b) ? number(b) : 0;
}
int blocks_excess(int dev, unsigned long long budget) {
  Block b;
  return g_store->excess(dev, budget, over, b) ? number(b) : 0;
}
int blocks_drop(int dev) {
  Block b;
  return g_store->drop(dev, b) ? number(b) : 0;
}
unsigned long long blocks_budget(unsigned long long free_b, unsigned long long total_b) {
  return keep_budget(free_b, total_b);
}
unsigned long long blocks_idle_bytes(int dev) { return g_store->idle_bytes(dev); }

}  // extern "C"
