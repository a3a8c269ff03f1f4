// Loaded into the global scope before the HIP runtime: hipMalloc, hipHostMalloc and
// hipGraphInstantiate are counted and passed on, or (shim_refuse_pinned) pinned memory
// is refused as a system without any left would.
#include <dlfcn.h>
#include <link.h>

#include <cstddef>
#include <cstring>
#include <string>

static int mallocs, pinned, graphs, refuse;

static void* real(const char* name) {
  static std::string path;
  if (path.empty())
    dl_iterate_phdr(
        [](dl_phdr_info* i, size_t, void*) {
          if (!std::strstr(i->dlpi_name, "libamdhip64.so")) return 0;
          path = i->dlpi_name;
          return 1;
        },
        nullptr);
  return dlsym(dlopen(path.c_str(), RTLD_LAZY | RTLD_NOLOAD), name);
}

extern "C" {

int hipMalloc(void** p, size_t n) {
  static int (*f)(void**, size_t) = reinterpret_cast<int (*)(void**, size_t)>(real("hipMalloc"));
  ++mallocs;
  return f(p, n);
}

int hipHostMalloc(void** p, size_t n, unsigned flags) {
  static int (*f)(void**, size_t, unsigned) = reinterpret_cast<int (*)(void**, size_t, unsigned)>(real("hipHostMalloc"));
  ++pinned;
  return refuse ? 2 : f(p, n, flags);  // 2: hipErrorOutOfMemory
}

int hipGraphInstantiate(void** exec, void* graph, void* node, char* log, size_t n) {
  static auto f = reinterpret_cast<int (*)(void**, void*, void*, char*, size_t)>(real("hipGraphInstantiate"));
  ++graphs;
  return f(exec, graph, node, log, n);
}

int shim_graphs() { return graphs; }
int shim_mallocs() { return mallocs; }
int shim_pinned() { return pinned; }
void shim_refuse_pinned(int on) { refuse = on; }
}
