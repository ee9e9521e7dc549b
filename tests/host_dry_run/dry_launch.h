// Test-only header, force-included when the library is compiled for a CPU dry run
// (tests/test_host_dry_run.py, tests/test_dispatch_host.py): a kernel launch only checks its geometry
// against the limits of the device (grid dimensions, threads per workgroup, LDS per workgroup; a violation
// traps) and reports success, so that the host code of every entry point (argument checks, workspace
// carving, launch planning) runs to its end on a machine without a GPU, under the compiler's
// undefined-behaviour checks.
// CIRC_DRY_DISPATCH: launches also note the kernel's name, and threads along x are held to the device's
// limit (the fuzzed shapes of the first test include many larger than any device memory).
#include <hip/hip_runtime.h>
#ifdef CIRC_DRY_DISPATCH
#include <typeinfo>
static char circ_dry_text[1 << 14];
static size_t circ_dry_used;
template <auto Kernel>
struct circ_dry_kernel {};
// one line per launch: the mangled name of a type that has the kernel, template arguments included, as its argument
template <auto Kernel>
static void circ_dry_note() {
  const char* s = typeid(circ_dry_kernel<Kernel>).name();
  if (circ_dry_used + 512 > sizeof(circ_dry_text)) return;
  while (*s && circ_dry_used + 2 < sizeof(circ_dry_text)) circ_dry_text[circ_dry_used++] = *s++;
  circ_dry_text[circ_dry_used++] = '\n';
  circ_dry_text[circ_dry_used] = 0;
}
extern "C" const char* circ_dry_log() { return circ_dry_text; }
extern "C" void circ_dry_clear() { circ_dry_text[circ_dry_used = 0] = 0; }
#define CIRC_DRY_NOTE(kern) circ_dry_note<(&kern)>()
#define CIRC_DRY_THREADS_X 4294967295ull
#else   // (naming the kernels instantiates them, which the first test has no use for)
#define CIRC_DRY_NOTE(kern) (void)0
#define CIRC_DRY_THREADS_X ~0ull
#endif
static inline void circ_dry_check(dim3 g, dim3 b, size_t lds) {
  const unsigned long long threads = (unsigned long long)b.x * b.y * b.z;
  if (g.x == 0 || g.y == 0 || g.z == 0 || g.x > 2147483647u || g.y > 65535u || g.z > 65535u || threads == 0 ||
      threads > 1024 || (unsigned long long)g.x * b.x > CIRC_DRY_THREADS_X || lds > 160u * 1024u)
    __builtin_trap();
}
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kern, grid, block, lds, stream, ...) \
  (CIRC_DRY_NOTE(kern), circ_dry_check(dim3(grid), dim3(block), size_t(lds)))
#define hipGetLastError() hipSuccess
#define hipFuncSetAttribute(...) hipSuccess
#define hipGetDevice(p) ((*(p) = 0), hipSuccess)
#define hipGetSymbolAddress(pp, sym) ((*(pp) = reinterpret_cast<void*>(0x7000000000ull)), hipSuccess)
