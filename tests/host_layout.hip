// What the host code of libpanda.so decides about sizes and layouts, printed
// for test_host_layout.py to check: no GPU, and no device memory behind the
// pointers.  usage: host_layout fold
#include <stdio.h>
#include <string.h>

#include "epilogues.h"
#include "host_internal.h"

using namespace panda;

// A product over k on packed C: the k of its first run, and its folding scratch.
static void fold() {
  using G = gemm::Tiles<3>::RectP;
  for (int64_t k = 16; k <= 4096; k += 16)
    printf("%lld %lld %zu\n", (long long)k, (long long)G::fold_run(k), rect_fold_floats(k, 3));
}

int main(int argc, char** argv) {
  if (argc != 2) return 2;
  if (!strcmp(argv[1], "fold")) fold();
  else return 2;
  return 0;
}
