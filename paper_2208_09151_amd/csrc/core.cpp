// Error reporting, the pinned blocks and version of the library (host only).
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <mutex>

#include "ginex.h"
#include "returns.hpp"

namespace ginex {

static thread_local char g_error[512] = "";

void set_error(const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof(g_error), fmt, ap);
  va_end(ap);
}

int32_t fail(int32_t code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_error, sizeof(g_error), fmt, ap);
  va_end(ap);
  return code;
}

// (kept until the process ends, when the runtime may be gone already)
static std::mutex g_block_mutex;
static void* g_free_blocks[HOST_BLOCKS];
static int g_free = 0, g_made = 0;

void* host_block_take() {
  const char* const pinned = getenv("GINEX_PINNED");
  if (pinned && pinned[0] == '0') return nullptr;
  int made;
  {
    std::lock_guard<std::mutex> lock(g_block_mutex);
    if (g_free > 0) return g_free_blocks[--g_free];
    if (g_made >= HOST_BLOCKS) return nullptr;
    made = ++g_made;
  }
  void* block = nullptr;
  if (hipHostMalloc(&block, HOST_BLOCK_BYTES, hipHostMallocPortable) == hipSuccess && block) {
    const char* const trace = getenv("GINEX_TRACE");
    if (trace && trace[0] == '2') fprintf(stderr, "[ginex] pinned block %d of at most %d\n", made, HOST_BLOCKS);
    return block;
  }
  (void)hipGetLastError();
  std::lock_guard<std::mutex> lock(g_block_mutex);
  --g_made;
  return nullptr;
}

void host_block_give(void* block) {
  std::lock_guard<std::mutex> lock(g_block_mutex);
  g_free_blocks[g_free++] = block;
}

}  // namespace ginex

extern "C" const char* ginex_last_error(void) { return ginex::g_error; }
extern "C" int32_t ginex_version(void) { return 10100; }
