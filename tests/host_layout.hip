// What the host code of libpanda.so decides about sizes and layouts, printed
// for test_host_layout.py to check: no GPU, and no device memory behind the
// pointers.  usage: host_layout fold | hpart | batch n Ne Na precision | small Ne Na |
// run Ne Na precision
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <vector>

#include "epilogues.h"
#include "host_internal.h"

using namespace panda;

// A product over k on packed C: the k of its first run, and its folding scratch.
static void fold() {
  using G = gemm::Tiles<3>::RectP;
  for (int64_t k = 16; k <= 4096; k += 16)
    printf("%lld %lld %zu\n", (long long)k, (long long)G::fold_run(k), rect_fold_floats(k, 3));
}

// The h partials that a load clears, and the room carved for them.
static void hpart() {
  const int64_t sizes[][2] = {{1, 2049},  {57, 4999}, {64, 18000}, {65, 2100}, {128, 5000},
                              {192, 900}, {320, 800}, {700, 18000}, {40, 400}, {500, 500}};
  static char base[256];
  for (const auto& s : sizes)
    for (int32_t prec : {PANDA_PREC_FP32, PANDA_PREC_BF16X3})
      for (int batched = 0; batched < 2; ++batched) {
        panda_ctx c{};
        ctx_layout(s[0], s[1], prec,
                   batched ? batch_spec(s[0], s[1]) : single_spec(s[0], s[1], false, prec), &c, base);
        const long long room = (char*)c.cstat - (char*)c.hpart;
        printf("%lld %lld %d %d %lld %lld\n", (long long)s[0], (long long)s[1], prec, batched,
               (long long)c.nh, room / 8);
      }
}

int main(int argc, char** argv) {
  if (argc == 6 && !strcmp(argv[1], "batch")) {  // whether n such networks take the small kernels
    const std::vector<int64_t> Ne(atoi(argv[2]), atoi(argv[3])), Na(atoi(argv[2]), atoi(argv[4]));
    printf("%d\n", (int)small_batch((int32_t)Ne.size(), Ne.data(), Na.data(), atoi(argv[5])));
    return 0;
  }
  if (argc == 4 && !strcmp(argv[1], "small")) {  // whether one network does
    printf("%d\n", (int)small_net(atoi(argv[2]), atoi(argv[3])));
    return 0;
  }
  if (argc == 5 && !strcmp(argv[1], "run")) {  // and whether it does when iterated alone
    printf("%d\n", (int)small_run(atoi(argv[2]), atoi(argv[3]), atoi(argv[4])));
    return 0;
  }
  if (argc != 2) return 2;
  if (!strcmp(argv[1], "fold")) fold();
  else if (!strcmp(argv[1], "hpart")) hpart();
  else return 2;
  return 0;
}
