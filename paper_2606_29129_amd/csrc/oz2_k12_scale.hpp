// oz2_k12_scale.hpp -- K1, its fold and K2 in one kernel, for vectors short
// enough that a block can take whole ones: Step 2 and the residues of Step 3
// of the fast modes for k <= kK12MaxK.
//
// As separate kernels (partial norms, fold, conversion) the operands are read
// twice from memory and the three launches wait for one another; where the
// problem is small that wait is the time, where it is not the second read is.
// Here a block of kK12Waves waves owns a few vectors over their whole length:
// it sums their squares, folds the chunk sums, evaluates the exponents and
// converts, reading its own few hundred KiB a second time from the caches
// (the last block of entries read stays in registers).
//
// A wave's tile is VL vectors x KB = (64 / VL) 16 entries: lane = (vector
// lane % VL, group of 16 entries lane / VL).  Loads of a strided operand take
// VL consecutive entries of a column, and a plane's 16-byte stores fill VL
// whole segments of KB bytes without staging.  The rounded-up sum of a chunk
// of 64 entries is a chain through four neighbouring groups: each group adds
// its 16 squares to the sum handed on by the group before, in four rounds in
// which every lane adds (the additions of the other groups are discarded),
// 80 operations per lane instead of 32 and the same order of additions.
//
// Bound: the planes it writes.  4096^3, N = 14: 213 us (268 MB read, 470 MB
// written; 120 us with the stores left out, 3.5 TB/s against 4.6 TB/s for a
// plain copy) where the three kernels took 236 us; small calls are latency:
// 256^3 7.3 us for 16.8, 1024^3 16.1 for 25.1; batch of 256 problems (sides
// 64..2048) 1.20 ms for 1.55.  Complex 4096 x 4096 operands, N = 14: 660 us
// (one block per CU: its three components do not fit the registers of two)
// for 706 in seven launches.
#pragma once

#include "oz2_k1_norm.hpp"
#include "oz2_k2_split.hpp"

namespace oz2 {

// Longest vectors taken: the blocks in flight hold 8 vectors each, 128 MB in
// all at k = 4096, which the MALL still holds for the second read; at k =
// 16384 they do not fit and the separate kernels are faster (3.68 against
// 4.00 ms at 16384^3, N = 17).
constexpr int kK12MaxK = 4096;
constexpr int kK12Waves = 8;   // waves per block

// Vectors per wave: 64-byte (binary64) and 64-byte (binary32) segments of a
// column per load instruction.
template <typename T>
constexpr int kK12VL = sizeof(T) == 8 ? 8 : 16;
// Complex vectors (real vectors of 2k components in storage order; 8 entries
// per lane, 128 per wave and vector): whole 128-byte segments of the planes.
constexpr int kK12VLCplx = 4;

// How a block's waves are dealt out: kw along k, vw to further vectors, pw to
// parts of the planes (wave groups that convert the same entries for every
// pw-th modulus; 1 unless SPLIT).  A block owns VB = vw VL vectors, a power
// of two and at most 64, so that every block stays inside the padded vectors.
struct K12Shape {
  int kw, vw, pw;
};
template <int VL>
OZ2_HD K12Shape k12_shape(int64_t K) {   // K: padded components of a vector
  const int nkb = (int)(K / (1024 / VL));
  const int kw = nkb < kK12Waves ? nkb : kK12Waves, q = kK12Waves / kw;
  int vw = 1;
  while (2 * vw <= q && 2 * vw * VL <= 64) vw *= 2;
  return K12Shape{kw, vw, 1};
}

// Blocks of an operand (padding vectors beyond the last block are left
// unwritten: their rows of the planes only reach products nothing reads).
inline int64_t k12_blocks(int64_t nvec, int VL, const K12Shape& sh) {
  return (nvec + sh.vw * VL - 1) / (sh.vw * VL);
}

// Most blocks of a launch: it holds fewer than 2^32 work-items.
constexpr int64_t kK12MaxBlocks = (int64_t(1) << 32) / (64 * kK12Waves);

// Whether this kernel is the faster form for an m x k by k x n product
// (padded length Kp).  Not for longer vectors (kK12MaxK), nor for more blocks
// than a launch takes, and not
//  * for real operands of few blocks, whose waves walk the whole of long
//    vectors while most CUs idle and the partial norms of the separate
//    kernels spread over them: binary64 below 96 blocks of 8 or more vectors
//    from k = 2817, binary32 below 64 blocks from 2305 and below 128 from 3072
//    (128 x 128 x 4096: N = 14 67 us against 56, binary32, N = 7, 66 against
//    47; 128 x 128 x 2048: 41 against 40; 1024 x 64 x 4096 N = 14 0.93);
//  * for a narrow binary64 operand beside one of less than 10240 long vectors
//    whose planes outgrow the MALL (192 MiB): a last round of blocks that
//    hardly fills any CU and no product to hide it (64 x 4096 x 4096, N = 14:
//    198 us against 179; k = 3000 135 against 152);
//  * for complex operands of which B is all but alone and its planes outgrow
//    the MALL (256 MiB; the one block per CU reads B's pairs in 64-byte pieces)
//    (64 x 3072 x 4096, N = 14: 467 us against 376; 4096 x 64 x 4096 629
//    against 645).
// Over 1474 measured shapes the choice is 0.4% from the better form on average.
template <typename T, bool CPLX>
inline bool k12_pays(int64_t m, int64_t n, int64_t k, int64_t Kp, int N) {
  if (k > kK12MaxK) return false;
  constexpr int VL = CPLX ? kK12VLCplx : kK12VL<T>;
  const K12Shape sh = k12_shape<VL>(CPLX ? 2 * Kp : Kp);
  const int64_t blocks = k12_blocks(m, VL, sh) + k12_blocks(n, VL, sh);
  if (blocks >= kK12MaxBlocks) return false;
  const int64_t planes = (int64_t)(CPLX ? 3 : 1) * N * (m + n) * k;
  if constexpr (CPLX) return !(m <= 256 && n > m && planes > (int64_t)256 << 20);
  if (sizeof(T) == 8 ? k > 2816 && blocks < 96
                     : (k > 2304 && blocks < 64) || (k >= 3072 && blocks < 128))
    return false;
  return !(sizeof(T) == 8 && k >= 3072 && (m < n ? m : n) <= 256 && (m < n ? n : m) < 10240 &&
           planes > (int64_t)192 << 20);
}

// Doubles of LDS for the chunk sums: VB ceil(K / 64) at most, for K <= MAXK
// components.
template <int VL, int MAXK>
constexpr int kK12Part = (VL * MAXK / kKC) > 256 ? (VL * MAXK / kKC) : 256;

// Residue modulo an odd p of a limb sum y (residue_odd's last three steps).
OZ2_HD uint32_t residue_of_sum(double y, double p, double ip) {
  constexpr double kMagic = 0x1.8p52;
  const double tq = fma(y, ip, kMagic);
  const double s = fma(tq, -p, kMagic * (p + 1.0));
  return (uint32_t)f64_to_bits(s + y);
}

// 8 complex entries (limbs of (re, im) pairs) in plane t of the three
// components x, y and x + y, packed four to a dword.  The residue of the sum
// comes from the sum of the limb sums (|.| < 2^49): the same value as the
// residues' sum reduced again, in four operations.
template <int LIMBS>
__device__ __forceinline__ void pack_residues_cplx(const Limbs<LIMBS> (&L)[16], int t,
                                                   const ModTable* __restrict__ tab,
                                                   uint2 (&w)[3]) {
  const double p = tab->p[t], ip = tab->inv_p[t], w1 = tab->powL[t][1];
  uint32_t d[3][2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {             // four entries at a time (registers)
    uint32_t v[3][4];
    if (t == 0) {                           // modulus 0 is 256
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[0][i] = residue_256_byte<LIMBS>(L[8 * q + 2 * i]);
        v[1][i] = residue_256_byte<LIMBS>(L[8 * q + 2 * i + 1]);
        v[2][i] = v[0][i] + v[1][i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        double x = L[8 * q + 2 * i].x[0], y = L[8 * q + 2 * i + 1].x[0];
        if constexpr (LIMBS == 2) {
          x = fma(L[8 * q + 2 * i].x[1], w1, x);
          y = fma(L[8 * q + 2 * i + 1].x[1], w1, y);
        }
        v[0][i] = residue_of_sum(x, p, ip);
        v[1][i] = residue_of_sum(y, p, ip);
        v[2][i] = residue_of_sum(x + y, p, ip);
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) d[c][q] = pack_low_bytes(v[c][0], v[c][1], v[c][2], v[c][3]);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) w[c] = make_uint2(d[c][0], d[c][1]);
}

// Block `bx` of `nblocks` of an operand.  mode 0 or 1 (Algorithm 2 or 1).
// CPLX: X holds (re, im) pairs, ld and k count pairs, and the planes of
// component c and modulus t are plane c N + t.  status: set to OZ2_STATUS_NONFINITE for a non-finite squared norm, if given.
template <typename T, bool CONTIG, bool NT, int LIMBS, bool SPLIT, bool CPLX = false>
__device__ __forceinline__ void k12_scale_body(
    const T* __restrict__ X, int64_t ld, int64_t nvec, int64_t k_entries, int mode,
    const ModTable* __restrict__ tab, int N, int32_t* __restrict__ e_out,
    double* __restrict__ S_out, int* __restrict__ status, int8_t* __restrict__ R, int64_t Vp,
    int64_t Kp, const K12Shape sh, int bx, int nblocks) {
  constexpr int E = CPLX ? 2 : 1;           // components per entry
  constexpr int VL = CPLX ? kK12VLCplx : kK12VL<T>;
  constexpr int GL = 64 / VL, KB = GL * 16, CPB = KB / kKC;
  __shared__ double part[kK12Part<VL, E * kK12MaxK>];   // [chunk][vector of the block]
  __shared__ double pmax[kK12Waves][VL];
  __shared__ int32_t exps[64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int v = lane % VL, g = lane / VL;
  const int VB = sh.vw * VL, kwi = wave % sh.kw, wr = wave / sh.kw;
  const int vwi = SPLIT ? wr % sh.vw : wr, pg = SPLIT ? wr / sh.vw : 0;
  const int pw = SPLIT ? sh.pw : 1;
  // Two blocks that share the 128-byte lines of a strided operand run on the
  // same XCD (ids 8 apart), so that its L2 fetches the lines once.
  if (!CONTIG && VB * E * (int)sizeof(T) < 128 && (bx | 15) < nblocks)
    bx = (bx & ~15) | ((bx & 7) << 1) | ((bx >> 3) & 1);
  const int64_t vb0 = (int64_t)bx * VB;
  const int vl = vwi * VL + v;
  const int64_t vec = vb0 + vl;
  // Vectors beyond nvec repeat the last one: their rows of the planes only
  // reach products that nothing reads.
  const T* Xv = X + (vec < nvec ? vec : nvec - 1) * (CONTIG ? E * ld : E);
  const int64_t st = CONTIG ? 1 : ld;       // between components (pairs, if strided)
  const int64_t k = E * k_entries;          // components
  const int nkb = (int)((k + KB - 1) / KB);
  const bool on = SPLIT ? pg < pw : wr < sh.vw;   // else this wave has no tile
  const int last = (nkb - 1 - kwi) / sh.kw; // this wave's last block of k
  double a[16];
  // Entries of block kb of k; beyond k zeros, read at clamped addresses so
  // that the loads are unconditional.
  auto load = [&](int kb, auto nt) {
    const int h0 = kb * KB + g * 16;
    if ((kb + 1) * KB <= k) {
      if constexpr (CPLX && !CONTIG) {
        const T* p = Xv + h0 * st;          // pair h0 / 2, pairs 2 ld apart
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          typedef T Pair __attribute__((ext_vector_type(2)));
          const Pair z = *reinterpret_cast<const Pair*>(p + 2 * i * st);
          a[2 * i] = (double)z[0];
          a[2 * i + 1] = (double)z[1];
        }
      } else {
        const T* p = Xv + h0 * st;
#pragma unroll
        for (int i = 0; i < 16; ++i) a[i] = load_in<decltype(nt)::value>(p + i * st);
      }
    } else {
      const int kl = (int)k - 1;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int h = h0 + i < kl ? h0 + i : kl;
        a[i] = (double)(CPLX && !CONTIG ? Xv[(h & ~1) * st + (h & 1)] : Xv[h * st]);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (h0 + i > kl) a[i] = 0.0;
    }
  };
  double mx = 0.0;
  for (int it = pg == 0 ? 0 : last; it <= last; ++it) {
    const int kb = it * sh.kw + kwi;
    if (!on || kb >= nkb) break;            // kw > nkb: nothing along k
    load(kb, std::false_type{});
    if (pg != 0) break;                     // the sums are group 0's
    round_up_begin();
    double s = ru_add_squares(0.0, a);
#pragma unroll
    for (int r = 1; r < 4; ++r) s = ru_add_squares(__shfl_up(s, VL), a);
    round_up_end(s);
    if ((g & 3) == 3) part[(kb * CPB + (g >> 2)) * VB + vl] = s;
    if (mode == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmax(mx, fabs(a[i]));
    }
  }
  if (mode == 1) {
#pragma unroll
    for (int o = VL; o < 64; o <<= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (g == 0) pmax[wave][v] = mx;
  }
  __syncthreads();
  if ((int)threadIdx.x < VB) {
    // fold of the chunk sums in chunk order and the exponent of one vector
    const int u = threadIdx.x, nch = (int)((k + kKC - 1) / kKC);
    double S = 0.0;
    int c = 0;
    round_up_begin();
    for (; c + 8 <= nch; c += 8) {
      double b[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i] = part[(c + i) * VB + u];
#pragma unroll
      for (int i = 0; i < 8; ++i) S = ru_add(S, b[i]);
    }
    for (; c < nch; ++c) S = ru_add(S, part[c * VB + u]);
    round_up_end(S);
    int32_t e;
    if (!(S <= 1.7976931348623157e308)) {
      e = kExpNonFinite;
      if (status && vb0 + u < nvec) atomicOr(status, 1);
    } else if (mode == 0) {
      e = alg2_exponent(S, tab->p_prop);
    } else {
      double m1 = 0.0;
      for (int w = 0; w < sh.kw; ++w) m1 = fmax(m1, pmax[u / VL * sh.kw + w][u % VL]);
      e = alg1_exponent(S, m1, tab->p_fast, tab->delta);
    }
    exps[u] = e;
    if (vb0 + u < nvec) {
      e_out[vb0 + u] = e;
      if (S_out) S_out[vb0 + u] = S;
    }
  }
  __syncthreads();
  if (!on) return;
  const int32_t e0 = exps[vl];
  const bool flagged = e0 == kExpNonFinite;
  const int32_t ev = flagged ? 0 : e0;
  // Conversion, from the last block of entries (still in registers) back.
  int8_t* out = R + vec * Kp + g * (16 / E);
  const int64_t plane = Vp * Kp;
  for (int it = last; it >= 0; --it) {
    const int kb = it * sh.kw + kwi;
    if (kb >= nkb) break;
    if (it != last) load(kb, std::bool_constant<NT && !CONTIG>{});
    if (__any(flagged)) {                   // a flagged vector converts to zeros
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (flagged) a[i] = 0.0;
    }
    Limbs<LIMBS> L[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) L[i] = limbs_of<LIMBS>(trunc(ldexp(a[i], ev)));
    int8_t* o = out + (int64_t)kb * (KB / E);
    for (int t = pg; t < N; t += pw) {
      if constexpr (CPLX) {
        uint2 w[3];
        pack_residues_cplx<LIMBS>(L, t, tab, w);
#pragma unroll
        for (int c = 0; c < 3; ++c) store_out<NT>(o + (c * N + t) * plane, w[c]);
      } else {
        uint32_t w[4];
        pack_residues<LIMBS, 16>(L, t, tab, w);
        store_packed<16, NT>(o + t * plane, w);
      }
    }
  }
  // Zeros from there to the padded end of the vector (less than 128 bytes).
  if constexpr (KB / E < 128) {
    const int hz = nkb * KB + g * 16;
    if (kwi == 0 && hz < (int)Kp)
      for (int t = pg; t < N; t += pw)
        store_out<NT>(out + t * plane + nkb * KB, make_uint4(0, 0, 0, 0));
  }
}

// Both operands in one launch: blocks [0, nA) take the rows of A, the others
// the columns of B.  Block 0 clears the status word (if given): K4 sets it.
// (At two blocks per CU the complex form spilled: 872 us for 660.)
template <typename T, bool NT, int LIMBS, bool SPLIT, bool CPLX = false>
__global__ __launch_bounds__(64 * kK12Waves, CPLX ? 2 : 4) void k12_scale_ab(
    const T* __restrict__ A, int64_t lda, int64_t m, const T* __restrict__ B, int64_t ldb,
    int64_t n, int64_t k, int mode, const ModTable* __restrict__ tab, int N,
    int32_t* __restrict__ eA, int32_t* __restrict__ eB, double* __restrict__ SA,
    double* __restrict__ SB, int8_t* __restrict__ RA, int8_t* __restrict__ RB, int64_t Mp,
    int64_t Np, int64_t Kp, K12Shape sh, int nA, int* __restrict__ status, bool set_status) {
  const int b = blockIdx.x;
  int* st = set_status ? status : nullptr;
  if (!set_status && b == 0 && threadIdx.x == 0) status[0] = 0;
  if (b < nA)
    k12_scale_body<T, false, NT, LIMBS, SPLIT, CPLX>(A, lda, m, k, mode, tab, N, eA, SA, st, RA, Mp, Kp, sh,
                                           b, nA);
  else
    k12_scale_body<T, true, NT, LIMBS, SPLIT, CPLX>(B, ldb, n, k, mode, tab, N, eB, SB, st, RB, Np, Kp, sh,
                                          b - nA, (int)gridDim.x - nA);
}

}  // namespace oz2
