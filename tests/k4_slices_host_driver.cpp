// Host build of K4's per-entry arithmetic with four slices whatever the
// table's own count (the instantiation of the batch's CRT kernel; test
// infrastructure): input and output as in k4_host_driver.cpp.  With an
// argument: the bound of the fast test for N = 2..kMaxN, as hex floats.
#define main k4_own_slices_main
#include "k4_host_driver.cpp"
#undef main

int main(int argc, char**) {
  static ModTable T;
  int N, E, U[kMaxN];
  if (argc > 1) {
    for (N = 2; N <= kMaxN; ++N) {
      if (!build_table(N, false, &T)) return 3;
      printf("%a\n", T.halfP);
    }
    return 0;
  }
  T.N = 0;
  while (scanf("%d %d", &N, &E) == 2) {
    if (N < 2 || N > kMaxN) return 2;
    if (T.N != N && !build_table(N, false, &T)) return 3;
    for (int t = 0; t < N; ++t)
      if (scanf("%d", &U[t]) != 1) return 4;
    one<kMaxSlices>(T, E, U);
  }
  return 0;
}
