// Host build of K4's per-entry arithmetic in the two forms that the kernels
// instantiate (test infrastructure): the table's own slice count with the
// two-slice test (plain, complex and fused kernels), and four slices whatever
// the table has (the batch's kernel).  Input as k4_host_driver.cpp; one line
// per case and form.  With an argument: per N = 2..kMaxN the bound of the fast
// test (hex float), the table's slices and the fused kernel's (0: none).
#define main k4_own_slices_main
#include "k4_host_driver.cpp"
#undef main
#include <utility>

#include "oz2_fused.hpp"

template <int S, bool OWN>
static void form(const ModTable& T, int E, const int* U) {
  double acc[S];
  for (int s = 0; s < S; ++s) acc[s] = 0.0;
  for (int t = 0; t < T.N; ++t)
    for (int s = 0; s < S; ++s) acc[s] = fma(T.w[t][s], (double)U[t], acc[s]);
  const double d = crt_unscale<S, 53, -1074, OWN>(acc, T, E);
  const float f = (float)crt_unscale<S, 24, -149, OWN>(acc, T, E);
  printf("%016llx %08x\n", (unsigned long long)f64_to_bits(d), (unsigned)f32_to_bits(f));
}

template <int... I>
static int fused_slices(int N, std::integer_sequence<int, I...>) {
  const int s[] = {fuse_slices(I)...};
  return N < (int)sizeof...(I) ? s[N] : 0;
}

int main(int argc, char**) {
  static ModTable T;
  int N, E, U[kMaxN];
  if (argc > 1) {
    for (N = 2; N <= kMaxN; ++N) {
      if (!build_table(N, false, &T)) return 3;
      printf("%a %d %d\n", T.halfP, T.slices,
             fused_slices(N, std::make_integer_sequence<int, kFuseMaxN + 1>()));
    }
    return 0;
  }
  T.N = 0;
  while (scanf("%d %d", &N, &E) == 2) {
    if (N < 2 || N > kMaxN) return 2;
    if (T.N != N && !build_table(N, false, &T)) return 3;
    for (int t = 0; t < N; ++t)
      if (scanf("%d", &U[t]) != 1) return 4;
    switch (T.slices) {
      case 1: form<1, true>(T, E, U); break;
      case 2: form<2, true>(T, E, U); break;
      case 3: form<3, true>(T, E, U); break;
      default: form<4, true>(T, E, U); break;
    }
    form<kMaxSlices, false>(T, E, U);
  }
  return 0;
}
