// oz2_fused.hpp -- K2 for the long operand, K3 and K4 in one kernel when the
// other operand is narrow: n <= 64 columns of B (the long operand is A, its
// rows strided) or m <= 64 rows of A (the long operand is B, its columns
// contiguous; the same product transposed).
//
// For a narrow operand the separate kernels are bound by memory: K2 writes N
// residue bytes per entry of the long operand, K3 reads them back once (a
// single row or column of tiles), and K4 reads the N product planes.  Here a
// workgroup owns 64 vectors of the long operand against all <= 64 of the
// narrow one and every modulus, 64 x 64 INT32 products per plane spread over
// the accumulators of 8 waves.  Per step of 64 k it
//   * converts its 64 x 64 entries (each once, 8 per lane; K2's arithmetic)
//     and writes the residues of all planes to LDS;
//   * multiplies them with the narrow operand's residues (made by K2
//     beforehand, brought to LDS during the conversion) on
//     v_mfma_i32_32x32x32_i8: wave w takes the 32 x 32 block w % 4 of the
//     planes of parity w / 4;
// and at the end reduces the products modulo p_t into LDS bytes, from which
// each lane reconstructs and unscales 8 outputs (K4's arithmetic).  No residue
// plane of the long operand and no product plane is stored.  The results are
// the separate kernels', bit for bit.
//
// Bound: the residues' arithmetic (about 4.75 N + 8 operations per entry).
// Two waves per SIMD (at most 128 accumulators each) rather than one with all
// moduli of 16 vectors: alone on its SIMD a wave issues an operation at best
// every 5.3 cycles, and a dependent binary64 one every 11 (two waves: 5.9).
// 65536 x 64 x 4096, N = 14: 1.06 ms (1.28 with one wave per SIMD), 2.15 GB
// read at 2.0 TB/s; the transposed shape 1.07 ms (2.0 ms in the separate
// kernels).  At N = 15 and 16 the accumulators leave too few registers: up to
// 18 dwords per lane spill at N = 15 and 5 at N = 16 (strided operand), none
// below.  With two moduli the loads are the bound, and one step of them in
// flight is little: the whole 12288 x 64 x 4096 call takes 196 us, 180 with the
// kernel of one wave per SIMD (N = 3: 1.03 at most; from 4 on faster).
#pragma once

#include <algorithm>
#include <utility>

#include "oz2_k1_norm.hpp"
#include "oz2_k2_split.hpp"
#include "oz2_k3_gemm.hpp"
#include "oz2_k4_crt.hpp"

namespace oz2 {

constexpr int kFuseCols = 64;   // vectors of the narrow operand
constexpr int kFuseMaxN = 16;   // moduli: accumulators and LDS
constexpr int kFuseK = 64;      // k per step
constexpr int kFuseRows = 64;   // vectors of the long operand per workgroup
constexpr int kFuseThreads = 512;
// Whether this kernel pays for `vecs` long vectors with k entries of `item`
// bytes.  It runs one block of 64 vectors per CU, and a round of 256 blocks
// takes the same time however few there are, so what counts is the part of
// the rounds that is filled.  From three quarters it wins over the separate
// kernels throughout (12288 x 64, N = 14: k = 256 0.95 of their time, 1024
// 0.80, 4096 0.58); below, from a length k whose planes cost them more, the
// longer the emptier the round (a single step of k is cheap from 9216 on):
//   8192 x 64, N = 14: k = 1024 1.31, 2048 0.95, 4096 0.77; binary32, N = 7:
//   k = 2048 1.17, 4096 0.79; 10240 x 64, N = 14: k = 1024 0.97, 1536 0.77;
//   6144 x 64, N = 14: k = 4096 0.95, 8192 1.09.
// With a second round the first, full one counts too: 18432 x 64, N = 14, k =
// 512 1.24, 1024 0.96, 2048 0.83.  Two or three moduli cost the separate
// kernels less (10240 x 64, N = 2: k = 2048 1.04, 4096 0.91).  Over 1792
// measured shapes (4096 to 32768 vectors, k = 64 to 16384, N = 2 to 16, both
// orientations) the rule is 0.9% from the better of the two on average.
inline bool fuse_pays(int64_t vecs, int64_t k, size_t item, int N) {
  const int64_t round = 256 * kFuseRows, rounds = (vecs + round - 1) / round;
  const double filled = (double)vecs / (double)(rounds * round);
  if (k <= kFuseK) return filled >= 0.5625;
  const double per_byte = (N < 4 ? 2.0 : 1.0) / ((double)k * (double)item);
  const double need = rounds == 1 ? 0.25 + 4096.0 * per_byte : 0.375 + 1536.0 * per_byte;
  return filled >= std::min(0.75, std::max(0.4375, need));
}

// 16-byte chunk position of logical k chunk g in the LDS row of vector c
// (rows of 64 bytes): spreads the 16-byte fragment reads, and the 8-byte
// writes of the converted residues, of 16 consecutive vectors over all banks.
__device__ __forceinline__ int fuse_swz(int c, int g) { return g ^ ((c >> 2) & 3); }

// Number of 39-bit CRT slices for the first NP moduli (P < 2^128 for NP <= 16),
// as the host tables compute it.
constexpr int fuse_slices(int NP) {
  unsigned __int128 P = 1;
  for (int t = 0; t < NP; ++t) P *= (unsigned)kModuli[t];
  int bits = 0;
  while (P) { ++bits; P >>= 1; }
  return (bits + kSliceBits - 1) / kSliceBits;
}

// 2^40 mod p (the weight of the high limb) and RN(1/p), as the host tables
// compute them, at compile time: the moduli of the fused kernel are template
// constants, so their constants need no table loads in the inner loop.
constexpr double fuse_pow40(int p) {
  unsigned long long r = 1;
  for (int i = 0; i < kLimbBits; ++i) r = (r * 2) % (unsigned long long)p;
  return (double)r;
}

constexpr double kFuseMagic = 0x1.8p52;

// 8 bytes per lane to LDS address a + off.  As asm, since the compiler
// cannot tell these writes from the direct global->LDS loads in flight to
// the other array and would wait for them first; the caller waits (lgkmcnt)
// before the barrier.  It fixes the place of the code behind it, five in six of
// whose instructions are 8 bytes long: left to chance (385 of 551 off by 4 in
// one build) the kernel took 2% more.  With two limbs a plane's code has an even
// number of 4-byte instructions up to its first long run, with one limb an odd
// one, hence the s_nop (65536 x 64 x 2048: N = 13 648 us without it, 629 with;
// N = 14, transposed, x 4096 1090 -> 1068).
template <int OFF, int LIMBS>
__device__ __forceinline__ void lds_write8(uint32_t a, uint32_t lo, uint32_t hi) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
  const u2 w = {lo, hi};
  if constexpr (LIMBS == 1)
    asm volatile(".p2align 3\n\ts_nop 0\n\tds_write_b64 %0, %1 offset:%2" ::"v"(a), "v"(w), "n"(OFF)
                 : "memory");
  else
    asm volatile(".p2align 3\n\tds_write_b64 %0, %1 offset:%2" ::"v"(a), "v"(w), "n"(OFF)
                 : "memory");
#endif
}
// The value is computed here, not later.
__device__ __forceinline__ void fuse_pin(double& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
}
template <int N>
__device__ __forceinline__ void wait_vmem_n_lds_all() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
#endif
}

template <typename F, int... I>
__device__ __forceinline__ void fuse_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, t>) for t = 0 .. NP-1, in order.
template <int NP, typename F>
__device__ __forceinline__ void fuse_for(F&& f) {
  fuse_for_impl(f, std::make_integer_sequence<int, NP>{});
}

// |a'| < 2^51 for the first 13 moduli (P < 2^103): one limb, no fold.
template <int NP>
constexpr int kFuseLimbs = NP <= 13 ? 1 : 2;

// Residue of a' for modulus index t, in the low byte of the result (what the
// packing reads): as residue_256_byte / residue_odd with the table values of
// modulus t.  One limb: |a'| < 2^51, so the quotient's error |a' / p| 2^-53 <
// 2^-2 / p stays below the 1 / (2p) distance from a half-integer, and
// 1.5 2^52 - q p stays in the binade of 1.5 2^52.
template <int t, int LIMBS>
__device__ __forceinline__ uint32_t fuse_residue(const Limbs<LIMBS>& L) {
  if constexpr (t == 0) {
    return residue_256_byte<LIMBS>(L);
  } else {
    constexpr double p = (double)kModuli[t], ip = 1.0 / (double)kModuli[t];
    double y = L.x[0];
    if constexpr (LIMBS == 2) y = fma(L.x[1], sconst(fuse_pow40(kModuli[t])), y);
    const double tq = fma(y, sconst(ip), kFuseMagic);
    const double s = fma(tq, sconst(-p), kFuseMagic * (p + 1.0));
    return (uint32_t)f64_to_bits(s + y);
  }
}

// Limbs of trunc(a 2^e) for this kernel, whose residues of the long operand
// are never stored.  A vector with a non-finite entry (exponent sentinel)
// gets a very negative exponent instead, so that its finite entries truncate
// to 0, and every value is clamped (infinities; NaNs too, since the minimum
// and maximum return the operand that is not a NaN): its residues are
// well-defined integers, and its outputs are NaN whatever its products are.
// For every other vector |a'| is below the clamp (P < 2^128 for N <= 16).
template <int LIMBS>
__device__ __forceinline__ Limbs<LIMBS> fuse_limbs(double a, int32_t e) {
  constexpr double kClamp = LIMBS == 1 ? 0x1p50 * 1.999 : 0x1p78;
  const double v =
      __builtin_fmin(__builtin_fmax(trunc(ldexp(a, e)), sconst(-kClamp)), sconst(kClamp));
  Limbs<LIMBS> L;
  if constexpr (LIMBS == 1) {
    L.x[0] = v;
  } else {
    L.x[1] = trunc(v * 0x1p-40);
    L.x[0] = fma(-L.x[1], 0x1p40, v);
  }
  return L;
}

// X: the long operand, entry h of vector v at X[v + h ld] or (CONTIG)
// X[v ld + h]; nx vectors, exponents eX.  RW: the narrow operand's residue
// planes (kFuseCols rows of Kp bytes each), nw vectors, exponents eW.  Output
// (x, w) at C[x + w ldc] or (CONTIG) C[w + x ldc].  NP = N, a template
// parameter: the moduli and their constants are compile-time values, and
// every accumulator access is unconditional.
template <typename T, typename TO, int NP, bool CONTIG>
__global__ __launch_bounds__(kFuseThreads, 2) void k234_fused(
    const T* __restrict__ X, int64_t ld, int64_t nx, int64_t nw, int64_t k,
    const int32_t* __restrict__ eX, const int32_t* __restrict__ eW,
    const int8_t* __restrict__ RW, int64_t Kp, const ModTable* __restrict__ tab,
    TO* __restrict__ C, int64_t ldc) {
  static_assert(NP >= 2 && NP <= kFuseMaxN, "moduli");
  constexpr int S = fuse_slices(NP), LIMBS = kFuseLimbs<NP>;
  constexpr int HP = (NP + 1) / 2;                   // planes per wave
  constexpr int PB = 64 * kFuseK;                    // bytes per plane and step
  __shared__ __attribute__((aligned(16))) int8_t ldsX[NP * PB];
  __shared__ __attribute__((aligned(16))) int8_t ldsW[NP * PB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t x0 = (int64_t)blockIdx.x * kFuseRows;

  // Conversion: this lane's vector xl and its 8 entries from kc of a step (a
  // wave reads 64 entries of a column of a strided operand, or 8 rows of 64
  // entries of a contiguous one).
  const int xl = CONTIG ? wave * 8 + (lane >> 3) : lane;
  const int kc = CONTIG ? (lane & 7) * 8 : wave * 8;
  const int64_t xv = x0 + xl;
  const bool xok = xv < nx;
  // vectors beyond nx convert to zero through the non-finite sentinel (their
  // outputs are never written)
  const int32_t e0 = xok ? eX[xv] : kExpNonFinite;
  const int32_t ex = e0 == kExpNonFinite ? -2000 : e0;   // see fuse_limbs
  const T* Xp = X + (xok ? xv : nx - 1) * (CONTIG ? ld : 1);
  const int64_t st = CONTIG ? 1 : ld;
  typedef __attribute__((address_space(3))) int8_t LdsByte;
  const uint32_t xdst = (uint32_t)(uintptr_t)(LdsByte*)(ldsX + xl * kFuseK +
                                                        fuse_swz(xl, kc >> 4) * 16 + (kc & 8));
  // The fewest load instructions load_x can take (16 bytes each at most): so
  // many may still be in flight when the narrow operand's slab is needed.
  constexpr int kXLoads = CONTIG ? 8 * (int)sizeof(T) / 16 : 8;
  double raw[8];
  // Only the last steps can run past k: there out-of-range k reads the last
  // entry (in bounds) and the value is zeroed when used.
  auto load_x = [&](int64_t k0) {
    const int64_t kb = k0 + kc;
    if (k0 + kFuseK <= k) {
      const T* p = Xp + kb * st;
      if constexpr (CONTIG) {
        constexpr int V = 16 / sizeof(T);
        typedef T Piece __attribute__((ext_vector_type(V), aligned(sizeof(T))));
#pragma unroll
        for (int i = 0; i < 8 / V; ++i) {
          const Piece q = *reinterpret_cast<const Piece*>(p + i * V);
#pragma unroll
          for (int j = 0; j < V; ++j) raw[i * V + j] = (double)q[j];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) raw[j] = load_in<true>(p + j * st);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) raw[j] = (double)Xp[(kb + j < k ? kb + j : k - 1) * st];
    }
  };
  // Narrow operand, half of the planes per 256 lanes: lane fills LDS slot
  // tid % 256 of a plane (vector / 4, stored chunk % 4, the swizzle being an
  // involution).
  const int wrow = (tid & 255) >> 2, whalf = (wave >> 2) & 1;
  const int64_t woff = (int64_t)wrow * Kp + fuse_swz(wrow, tid & 3) * 16;
  auto load_w = [&](int64_t k0) {
#pragma unroll
    for (int t = 0; t < HP; ++t)
      if (2 * t + whalf < NP)
        load_lds16(RW + (int64_t)(2 * t + whalf) * kFuseCols * Kp + woff + k0,
                   ldsW + (2 * t + whalf) * PB + (wave & 3) * 64 * 16);
  };

  const int bx = (wave >> 1) & 1, bw = wave & 1, half = (wave >> 2) & 1;
  v16i acc[HP];
#pragma unroll
  for (int t = 0; t < HP; ++t) acc[t] = v16i{0};

  const int nsteps = (int)((k + kFuseK - 1) / kFuseK);
  load_x(0);
  for (int s = 0; s < nsteps; ++s) {
    const int64_t k0 = (int64_t)s * kFuseK;
    if (k0 + kc + 8 > k) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (k0 + kc + j >= k) raw[j] = 0.0;
    }
    Limbs<LIMBS> L[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) L[j] = fuse_limbs<LIMBS>(raw[j], ex);
    // the entries are in, and used, before more loads go out (a wait for them
    // behind those would wait for those too)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < LIMBS; ++i) fuse_pin(L[j].x[i]);
    __builtin_amdgcn_sched_barrier(0);
    load_w(k0);                          // lands during the conversion
    if (s + 1 < nsteps) load_x(k0 + kFuseK);
    fuse_for<NP>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      lds_write8<t * PB, LIMBS>(
          xdst,
          pack_low_bytes(fuse_residue<t>(L[0]), fuse_residue<t>(L[1]), fuse_residue<t>(L[2]),
                         fuse_residue<t>(L[3])),
          pack_low_bytes(fuse_residue<t>(L[4]), fuse_residue<t>(L[5]), fuse_residue<t>(L[6]),
                         fuse_residue<t>(L[7])));
      __builtin_amdgcn_sched_barrier(0);   // one plane at a time (registers)
    });
    // the narrow operand's slab of this step has landed (the next entries of
    // the long one may still be on their way; binary32 ones are waited for
    // where they are converted, behind their loads)
    if (s + 1 < nsteps) wait_vmem_n_lds_all<kXLoads>();
    else wait_vmem_lds_all();
    __syncthreads();
#pragma unroll
    for (int t = 0; t < HP; ++t) {
      if (2 * t + half < NP) {
        const int8_t* px = ldsX + (2 * t + half) * PB;
        const int8_t* pw = ldsW + (2 * t + half) * PB;
        const int rx = bx * 32 + (lane & 31), rw = bw * 32 + (lane & 31);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int g = kk * 2 + (lane >> 5);
          const v4i fx = *reinterpret_cast<const v4i*>(px + rx * kFuseK + fuse_swz(rx, g) * 16);
          const v4i fw = *reinterpret_cast<const v4i*>(pw + rw * kFuseK + fuse_swz(rw, g) * 16);
          acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fx, fw, acc[t], 0, 0, 0);
        }
      }
    }
    __syncthreads();       // every wave is done with this step's slabs
  }

  // Epilogue: the residues of the products as bytes in LDS, plane by plane
  // [vector along the contiguous side of C][other vector], in ldsX.
#pragma unroll
  for (int t = 0; t < HP; ++t) {
    if (2 * t + half < NP) {
      const int tt = 2 * t + half;
      const double p = tab->p[tt], ip = tt == 0 ? 0.0 : tab->inv_p[tt];  // 256: the low byte
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rx = bx * 32 + acc_row(r, lane), rw = bw * 32 + acc_col(lane);
        ldsX[tt * PB + (CONTIG ? rw * 64 + rx : rx * 64 + rw)] =
            (int8_t)residue_sym_i32(acc[t][r], p, ip);
      }
    }
  }
  __syncthreads();
  // Lane = the vector along C's columns; outputs 8 wave .. 8 wave + 7 across.
  double sums[8][S];
#pragma unroll
  for (int j = 0; j < 8; ++j)
#pragma unroll
    for (int q = 0; q < S; ++q) sums[j][q] = 0.0;
  for (int t = 0; t < NP; ++t) {
    const uint2 b = *reinterpret_cast<const uint2*>(ldsX + t * PB + lane * 64 + wave * 8);
    double wt[S];
#pragma unroll
    for (int q = 0; q < S; ++q) wt[q] = tab->w[t][q];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const double u = (double)(int)(int8_t)((j < 4 ? b.x : b.y) >> (8 * (j & 3)));
#pragma unroll
      for (int q = 0; q < S; ++q) sums[j][q] = fma(wt[q], u, sums[j][q]);
    }
  }
  const ModTable& TB = *tab;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int xi = CONTIG ? wave * 8 + j : lane, wi = CONTIG ? lane : wave * 8 + j;
    const int64_t x = x0 + xi;
    if (x < nx && wi < nw) {
      const int32_t e = eX[x], f = eW[wi];
      double v;
      if (e == kExpNonFinite || f == kExpNonFinite) v = __builtin_nan("");
      else if constexpr (sizeof(TO) == 8) v = crt_unscale<S, 53, -1074, true>(sums[j], TB, e + f);
      else v = crt_unscale<S, 24, -149, true>(sums[j], TB, e + f);
      C[CONTIG ? wi + x * ldc : x + wi * ldc] = (TO)v;
    }
  }
}

}  // namespace oz2
