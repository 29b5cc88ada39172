// Host build of the rules that choose a call's kernels (test infrastructure):
// reads "k12 TYPE m n k N" or "fuse TYPE vecs k N" from stdin (TYPE d, s, z or
// c), prints 0 or 1 per line.
#include <cstdio>
#include <cstring>

#include "oz2_fused.hpp"
#include "oz2_k12_scale.hpp"

using namespace oz2;

int main() {
  char what[8], type[4];
  while (scanf("%7s %3s", what, type) == 2) {
    long long a, b, c;
    int N;
    if (!strcmp(what, "fuse")) {
      if (scanf("%lld %lld %d", &a, &b, &N) != 3) return 2;
      printf("%d\n", (int)fuse_pays(a, b, type[0] == 'd' ? 8 : 4, N));
      continue;
    }
    if (scanf("%lld %lld %lld %d", &a, &b, &c, &N) != 4) return 2;
    const int64_t Kp = (c + 127) / 128 * 128;
    printf("%d\n", (int)(type[0] == 'd'   ? k12_pays<double, false>(a, b, c, Kp, N)
                         : type[0] == 's' ? k12_pays<float, false>(a, b, c, Kp, N)
                         : type[0] == 'z' ? k12_pays<double, true>(a, b, c, Kp, N)
                                          : k12_pays<float, true>(a, b, c, Kp, N)));
  }
  return 0;
}
