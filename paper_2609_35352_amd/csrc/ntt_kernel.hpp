// Negacyclic NTT passes for gfx950 and the rescale epilogue built on them.
//
// Convention (the NTT domain the library's ciphertexts live in):
//     a_hat_k = sum_n a_n psi^((2k+1) n)  mod q,   k = 0 .. N-1 in natural order,
// psi a primitive 2N-th root of unity mod q.  With omega = psi^2 this is the
// cyclic DFT of the twisted sequence a_n psi^n; its inverse is
//     a_n = N^-1 psi^-n sum_k a_hat_k omega^(-nk).
//
// Both run as a four-step transform, N = N1 * N2 (256 x 256 for N = 2^16):
// index n = n1 + N1 n2 on the input side and k = k2 + N2 k1 on the output
// side, so that omega^(nk) = omega^(n1 k2) (omega^N2)^(n1 k1) (omega^N1)^(n2 k2).
//   pass A: for each n1, a transform of size N2 over n2, then a multiplication
//           by mid (n1, k2); stored as row k2 of the intermediate, column n1;
//   pass B: for each k2, a DFT of size N1 over n1, giving output k2 + N2 k1
//           (inverse: multiplied by post[k1]).
// Forward, pass A's transform is itself negacyclic: with phi = psi^N1 it takes
// x_n2 to sum x_n2 phi^((2 k2 + 1) n2), by butterflies a + t b, a - t b with
// t = phi^bitrev(2^s + block) (stage s from the largest distance down, input
// natural, output bit-reversed): the twist psi^(N1 n2) rides in the
// butterflies' twiddles, and psi^n1, constant along the transform, in mid.
// Inverse, pass A's transform is the cyclic DFT, and the factor N^-1 psi^-k
// splits into a part constant along pass B's DFT, in mid, and post.  The cyclic
// DFTs are radix 2 with the input in bit-reversed order and the output natural.
// A workgroup takes kNttCols columns (pass A) or rows (pass B) at once, so
// every global access is a run of at least kNttCols consecutive words.  A
// thread takes groups of up to 16 words through four stages at a time in
// registers, and LDS carries the data between groups.
//
// Arithmetic is in fp64, on exact integers (q < 2^50): a double holds any
// integer below 2^53, and gfx950 issues fp64 FMA at full rate where 32-bit
// integer multiplies run at quarter rate.  A modular product b * w follows the
// FMA method of van der Hoeven, Lecerf and Quintin ("Modular SIMD arithmetic in
// Mathemagix", 2016): h = fl(b w) and its exact error l = b w - h (one FMA);
// the quotient k = rint(b * w/q) from one FMA against a rounding constant;
// then b w - k q = (h - k q) + l exactly.  The tables hold centred twiddles,
// |w| <= q/2: then for |b| < 2^52 the quotient stays below 2^51 and the result
// r satisfies r = b w (mod q) and |r| <= q (1/2 + |b| 2^-54).  Values between
// stages are signed and lazily reduced (BoundsTransform checks every bound at
// compile time, of the passes' groups of stages and of the whole transforms'); reduce() brings any |x| < 2^53 to |x| <= q/2 + 1, and any
// |x| < 2^52 to the exact centred residue, |x| <= (q-1)/2 (the FMA's error
// |x/q| 2^-53 is then below 1/(2q), the distance from x/q to the nearest
// half-integer).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "buffer.hpp"

namespace fiona {

constexpr uint32_t kNttCols = 16;      // columns (pass A) or rows (pass B) per workgroup
constexpr uint32_t kNttThreads = 256;

struct Tw {   // a twiddle w, an integer with |w| <= q/2, and fl(w / q)
  double w, wq;
};

// 1.5 * 2^52: adding it to |v| < 2^51 rounds v to the nearest integer.
constexpr double kRound = 6755399441055744.0;

__device__ __forceinline__ double mul_tw(double b, const Tw &t, double q) {
#pragma clang fp contract(off)
  const double h = b * t.w;
  const double l = __builtin_fma(b, t.w, -h);
  const double k = __builtin_fma(b, t.wq, kRound) - kRound;
  return __builtin_fma(-k, q, h) + l;
}

__device__ __forceinline__ double reduce(double x, double q, double qinv) {
#pragma clang fp contract(off)
  const double k = __builtin_fma(x, qinv, kRound) - kRound;
  return __builtin_fma(-k, q, x);
}

// x an integer, |x| < 2^52 -> its residue in [0, q)
__device__ __forceinline__ double canonical(double x, double q, double qinv) {
  const double z = reduce(x, q, qinv);
  return z < 0.0 ? z + q : z;
}

// Integers below 2^52 to and from doubles: 2^52 + x has the bits of x in its
// mantissa, so the conversion is one bitwise operation and one exact add.
__device__ __forceinline__ double to_f64(uint64_t x) {   // x < 2^52
  return __builtin_bit_cast(double, x | 0x4330000000000000ull) - 4503599627370496.0;
}
__device__ __forceinline__ uint64_t to_u64(double y) {   // y an integer in [0, 2^52)
  return __builtin_bit_cast(uint64_t, y + 4503599627370496.0) & 0x000FFFFFFFFFFFFFull;
}

// A buffer view of global memory for the passes' per-group accesses.  The
// descriptor holds the base and the bytes left in the buffer; the byte
// offset splits into the lane's part (a VGPR) and a part the workgroup
// shares (an SGPR or a constant), so that the 16 accesses of a group need no
// vector address arithmetic.  Offsets stay below 2^32 bytes (one vector or
// one table per view).
typedef uint32_t nv2 __attribute__((ext_vector_type(2)));
typedef uint32_t nv4 __attribute__((ext_vector_type(4)));
struct Buf {
  __amdgpu_buffer_rsrc_t rs;
  // p is the same in every lane; readfirstlane keeps the descriptor in SGPRs
  // where the compiler has computed p in vector registers.  end: the end of
  // the buffer p points into.
  __device__ __forceinline__ Buf(const void *p, const void *end) : rs(make(p, end)) {}
  static __device__ __forceinline__ __amdgpu_buffer_rsrc_t make(const void *p, const void *end) {
    const uint64_t a = (uint64_t)p;
    // readfirstlane returns an int; join_halves takes it as unsigned
    const uint64_t u = join_halves((uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)),
                                   (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a));
    return __builtin_amdgcn_make_buffer_rsrc((void *)u, (short)0, (int)buffer_extent(u, (uint64_t)end), 0x00020000);
  }
  __device__ __forceinline__ uint64_t u64(uint32_t voff, uint32_t soff) const {
    const nv2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0);
    return (uint64_t)w.x | ((uint64_t)w.y << 32);
  }
  __device__ __forceinline__ double f64(uint32_t voff, uint32_t soff) const {
    return __builtin_bit_cast(double, u64(voff, soff));
  }
  // Nontemporal loads (cache policy 2) for words read once: pass B's
  // intermediate and the words it subtracts from.
  __device__ __forceinline__ uint64_t u64_once(uint32_t voff, uint32_t soff) const {
    const nv2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 2);
    return (uint64_t)w.x | ((uint64_t)w.y << 32);
  }
  __device__ __forceinline__ double f64_once(uint32_t voff, uint32_t soff) const {
    return __builtin_bit_cast(double, u64_once(voff, soff));
  }
  __device__ __forceinline__ Tw tw(uint32_t voff, uint32_t soff) const {
    const nv4 w = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0);
    return Tw{__builtin_bit_cast(double, (uint64_t)w.x | ((uint64_t)w.y << 32)),
              __builtin_bit_cast(double, (uint64_t)w.z | ((uint64_t)w.w << 32))};
  }
  // Stores of the callers' words are nontemporal (cache policy 2).
  __device__ __forceinline__ void put(uint64_t x, uint32_t voff, uint32_t soff) const {
    __builtin_amdgcn_raw_buffer_store_b64((nv2){(uint32_t)x, (uint32_t)(x >> 32)}, rs, voff, soff, 2);
  }
  // Stores of intermediates and remainders, nontemporal or with the default
  // policy (stores_nontemporal in ntt_host.hpp).
  template <bool NT>
  __device__ __forceinline__ void put(double y, uint32_t voff, uint32_t soff) const {
    const uint64_t x = __builtin_bit_cast(uint64_t, y);
    __builtin_amdgcn_raw_buffer_store_b64((nv2){(uint32_t)x, (uint32_t)(x >> 32)}, rs, voff, soff, NT ? 2 : 0);
  }
};

__host__ __device__ constexpr uint32_t bit_reverse(uint32_t x, uint32_t bits) {
  return __builtin_bitreverse32(x) >> (32 - bits);
}
// The four-bit reversal of u < 16 (a group's position in the bit-reversed order).
__host__ __device__ constexpr uint32_t rev4(uint32_t u) {
  return ((u & 1u) << 3) | ((u & 2u) << 1) | ((u & 4u) >> 1) | ((u & 8u) >> 3);
}

// LDS layout of the kNttCols columns.  The 16 lanes of a quarter wave work on
// the same word of 16 different columns (the DFT's twiddle reads are then
// broadcasts), so the column stride is odd: those lanes fall into 16
// different banks.  Within a column one padding word follows every 16, so
// that 16 consecutive bit-reversed positions (the row loads of pass B) fall
// into different banks too.
__host__ __device__ constexpr uint32_t pidx(uint32_t i) { return i + (i >> 4); }
__host__ __device__ constexpr uint32_t padded_len(uint32_t m) { return m + m / 16 + 1; }

// Stages S0 .. S0+R-1 of the radix-2 DFT on one group of 2^R words held in
// registers: r[u] is the word at position o + (u << S0) of a group whose
// offset below 2^S0 is o (positions in the DFT's bit-reversed input order).
// tw_at(t) returns w_M^t.  Nothing is reduced here but, in the first group
// (S0 = 0), the even words after its second stage: the butterflies with the
// twiddle 1 add their input unmultiplied, so those words double in both
// stages, while a product's output is back near q/2.  BoundsTransform follows every
// word's bound through this schedule.  Reducing every word after every second
// stage instead took 8 reductions a word and transform pair, now 3.  That alone
// left the large rescales as they were (1.07 ms at N = 2^16, L = 8, 128
// ciphertexts: the passes wait on memory there) and made small ones 4% faster
// (N = 2^14, L = 6, 24 ciphertexts: 46.9 -> 45.0 us).
template <uint32_t LOGM, uint32_t S0, uint32_t R, typename TwAt>
__device__ __forceinline__ void butterflies(double (&r)[1u << R], uint32_t o, TwAt tw_at, double q, double qinv) {
  constexpr uint32_t S = 1u << R;
#pragma unroll
  for (uint32_t st = 0; st < R; ++st) {
    const uint32_t hh = 1u << st, shift = LOGM - 1 - (S0 + st);
#pragma unroll
    for (uint32_t u0 = 0; u0 < S; ++u0) {
      if ((u0 & (2 * hh - 1)) >= hh) continue;
      // with S0 = 0 (so o = 0) the butterflies with offset 0 have the twiddle 1
      const bool unit = S0 == 0 && (u0 & (hh - 1)) == 0;
      const double a = r[u0];
      const double t = unit ? r[u0 + hh] : mul_tw(r[u0 + hh], tw_at((o + ((u0 & (hh - 1)) << S0)) << shift), q);
      r[u0] = a + t;
      r[u0 + hh] = a - t;
    }
    if (S0 == 0 && st == 1 && R > 2) {
#pragma unroll
      for (uint32_t u = 0; u < S; u += 2) r[u] = reduce(r[u], q, qinv);
    }
  }
}

// Stages S0 .. S0+R-1 of the negacyclic transform on one group of 2^R words at
// distance 2^(LOGM-S0-R) of each other inside block `block` of stage S0:
// tw_at(2^s + b) is the twiddle of block b of stage s.  Nothing is reduced.
template <uint32_t S0, uint32_t R, typename TwAt>
__device__ __forceinline__ void tree_butterflies(double (&r)[1u << R], uint32_t block, TwAt tw_at, double q) {
#pragma unroll
  for (uint32_t st = 0; st < R; ++st) {
    const uint32_t hh = 1u << (R - 1 - st);
#pragma unroll
    for (uint32_t b = 0; b < (1u << st); ++b) {
      const Tw t = tw_at((1u << (S0 + st)) + (block << st) + b);
#pragma unroll
      for (uint32_t k = 0; k < hh; ++k) {
        const uint32_t u0 = b * 2 * hh + k;
        const double a = r[u0], x = mul_tw(r[u0 + hh], t, q);
        r[u0] = a + x;
        r[u0 + hh] = a - x;
      }
    }
  }
}

// Bounds of the words through a transform of `stages` stages, the first `first`
// of them in a thread's first group, whose input is at most `in`, in units of
// 2^50 (every q is below one unit): a product's input must stay below 4 units
// and every word below 8 (exact integers in a double).  tree: the negacyclic
// transform (tree_butterflies), else the DFT (butterflies).  Both kinds reduce
// every word after the first group (put_first, tree_first, and the same in
// ntt_whole.hpp).
constexpr double kUnitReduced = 0.5 + 0x1p-40;   // after reduce(): at most q/2 + 1
constexpr double product_bound(double b) { return 0.5 + b / 16; }
struct BoundsTransform {
  bool ok = true;
  double out = 0;   // the last group's output
  constexpr double product(double b) {
    if (b >= 4) ok = false;
    return product_bound(b);
  }
  constexpr double word(double x) {
    if (x >= 8) ok = false;
    return x;
  }
  constexpr BoundsTransform(uint32_t stages, uint32_t first, double in, bool tree) {
    double r[16] = {};
    for (int u = 0; u < 16; ++u) r[u] = in;
    for (int st = 0; st < (int)first; ++st) {   // the first group
      const int hh = 1 << st;
      for (int u = 0; u < 1 << first; ++u) {
        if ((u & (2 * hh - 1)) >= hh) continue;
        const double t = !tree && (u & (hh - 1)) == 0 ? r[u + hh] : product(r[u + hh]);
        const double x = word(r[u] + t);
        r[u] = x;
        r[u + hh] = x;
      }
      if (!tree && st == 1 && first > 2)
        for (int u = 0; u < 16; u += 2) r[u] = kUnitReduced;
    }
    out = kUnitReduced;
    for (uint32_t st = first; st < stages; ++st) out = word(out + product(out));
  }
};
// The output of a transform of 2^stages words.  Inputs: residues, or pass A's
// products by mid, whose quotient takes w / q as w fl(1/q), twice the rounding
// error: 1/2 + b/8 of an input b below 4; forward, integers below 2^50.
template <uint32_t STAGES, uint32_t FIRST>
constexpr double transform_out() {
  constexpr BoundsTransform b(STAGES, FIRST, 1.0, false), t(STAGES, FIRST, 1.0, true);
  static_assert(b.ok && t.ok, "a product's input or a word passes its bound");
  static_assert(b.out < 4 && t.out < 4, "the products after the last stage (mid, post) take their input below 4 units");
  return b.out > t.out ? b.out : t.out;
}
template <uint32_t LOGM>
constexpr double dft_out() { return transform_out<LOGM, 4>(); }   // the passes': first groups of 16

// How a size-M DFT (M = 64 .. 512: kSideMinA .. kSideMaxB in ntt_host.hpp) splits over a workgroup's
// kNttCols columns.  The first four stages run on groups of 16 words that a
// thread loads straight from global memory (natural index i' + I1 v,
// v < 16: position 16 i + bitrev4(v) of the bit-reversed input order,
// i = bitrev(i') over log2(I1) bits); the last R2 stages run on groups of
// 2^R2 words (positions o + (u << S0L), o < I2) whose results, the outputs
// k = o + (u << S0L) in natural order, the thread stores straight to global
// memory; what lies between (M = 512: one stage) runs in LDS.
template <uint32_t LOGM>
struct DftShape {
  static constexpr uint32_t M = 1u << LOGM, PM = padded_len(M);
  static constexpr uint32_t I1 = M / 16;                       // first groups per column
  static constexpr uint32_t R2 = LOGM <= 8 ? LOGM - 4 : 4;      // stages of the last groups
  static constexpr uint32_t S0L = LOGM - R2;                   // the last groups' first stage
  static constexpr uint32_t E2 = 1u << R2, I2 = 1u << S0L;     // last group size and count per column
  static constexpr uint32_t IT1 = kNttCols * I1, IT2 = kNttCols * I2;
};

// The twiddles of the first four stages, w_M^(j M/16) for j < 8: uniform
// over the workgroup, read once into scalar registers.
template <uint32_t LOGM>
__device__ __forceinline__ void first_twiddles(Tw (&t1)[8], const Tw *__restrict__ dft) {
#pragma unroll
  for (uint32_t j = 0; j < 8; ++j) t1[j] = dft[j << (LOGM - 4)];
}

template <uint32_t LOGM>
__device__ __forceinline__ void first_stages(double (&r)[16], const Tw (&t1)[8], double q, double qinv) {
  butterflies<LOGM, 0, 4>(r, 0, [&](uint32_t t) { return t1[t >> (LOGM - 4)]; }, q, qinv);
}

// The first groups' results go to LDS, reduced: column col, group i' (natural order).
template <uint32_t LOGM>
__device__ __forceinline__ void put_first(double *xs, uint32_t col, uint32_t ip, const double (&r)[16], double q,
                                          double qinv) {
  using D = DftShape<LOGM>;
  const uint32_t i = bit_reverse(ip, LOGM - 4);
#pragma unroll
  for (uint32_t u = 0; u < 16; ++u) xs[col * D::PM + pidx(16 * i + u)] = reduce(r[u], q, qinv);
}

// The negacyclic transform's first groups: r[v] is row i' + I1 v.  They go to
// LDS, reduced: position v I1 + i' of column col.
template <uint32_t LOGM>
__device__ __forceinline__ void tree_first(double *xs, uint32_t col, uint32_t ip, double (&r)[16],
                                           const Tw *__restrict__ tree, double q, double qinv) {
  using D = DftShape<LOGM>;
  tree_butterflies<0, 4>(r, 0, [&](uint32_t t) { return tree[t]; }, q);
#pragma unroll
  for (uint32_t v = 0; v < 16; ++v) xs[col * D::PM + pidx(v * D::I1 + ip)] = reduce(r[v], q, qinv);
}

// Its last groups: on return r[e] is output o + (bitrev(e) << S0L), at most
// dft_out() units: positions j E2 + e of block j = bitrev(o).
template <uint32_t LOGM>
__device__ __forceinline__ void tree_last(const double *xs, uint32_t col, uint32_t o, const Tw *tw,
                                          double (&r)[DftShape<LOGM>::E2], double q) {
  using D = DftShape<LOGM>;
  const uint32_t j = bit_reverse(o, D::S0L);
#pragma unroll
  for (uint32_t e = 0; e < D::E2; ++e) r[e] = xs[col * D::PM + pidx(j * D::E2 + e)];
  tree_butterflies<D::S0L, D::R2>(r, j, [&](uint32_t t) { return tw[t]; }, q);
}

// Between the first and the last groups: the middle stages in LDS (M = 512),
// each thread taking groups of two in turn; barriers on both sides.
template <uint32_t LOGM>
__device__ __forceinline__ void middle_stages(double *xs, const Tw *tw, double q, double qinv) {
  using D = DftShape<LOGM>;
  __syncthreads();
  if constexpr (D::S0L > 4) {
    static_assert(D::S0L == 5, "one middle stage at most");
    for (uint32_t it = threadIdx.x; it < kNttCols * D::M / 2; it += kNttThreads) {
      const uint32_t col = it % kNttCols, gi = it / kNttCols, o = gi & 15u, base = ((gi >> 4) << 5) + o;
      double r[2] = {xs[col * D::PM + pidx(base)], xs[col * D::PM + pidx(base + 16)]};
      butterflies<LOGM, 4, 1>(r, o, [&](uint32_t t) { return tw[t]; }, q, qinv);
      xs[col * D::PM + pidx(base)] = r[0];
      xs[col * D::PM + pidx(base + 16)] = r[1];
    }
    __syncthreads();
  }
}

// The last groups: column col, offset o; on return r[u] is output o + (u << S0L), at most dft_out() units.
template <uint32_t LOGM>
__device__ __forceinline__ void last_stages(const double *xs, uint32_t col, uint32_t o, const Tw *tw,
                                            double (&r)[DftShape<LOGM>::E2], double q, double qinv) {
  using D = DftShape<LOGM>;
#pragma unroll
  for (uint32_t u = 0; u < D::E2; ++u) r[u] = xs[col * D::PM + pidx(o + (u << D::S0L))];
  butterflies<LOGM, D::S0L, D::R2>(r, o, [&](uint32_t t) { return tw[t]; }, q, qinv);
}

// b - y for a residue b and a transform's output y, small enough for a product:
// REDUCE, where y's bound does not leave room for b.
template <bool REDUCE>
__device__ __forceinline__ double minuend(uint64_t b, double y, double q, double qinv) {
  if constexpr (REDUCE) y = reduce(y, q, qinv);
  return to_f64(b) - y;
}
template <uint32_t LOGM>
constexpr bool reduce_minuend() { return dft_out<LOGM>() + 1 >= 4; }

// Copy n twiddles into LDS.
__device__ __forceinline__ void stage_twiddles(Tw *dst, const Tw *__restrict__ src, uint32_t n) {
  for (uint32_t i = threadIdx.x; i < n; i += kNttThreads) dst[i] = src[i];
}

// What a pass reads (pass A) and writes (pass B).  Natural order is the
// callers' layout.  The library's own vectors use layouts in which a
// workgroup's 16 columns or rows are contiguous:
//   transposed: element i = k2 + N2 k1 (k2 < N2, k1 < N1, the split of the
//     four-step transform's output) at k2 N1 + k1, so that one pass-B row k2
//     is N1 contiguous words;
//   blocked: element n = n1 + N1 n2 (the split of its input) at
//     ((n1 / 16) N2 + n2) 16 + n1 mod 16, so that one pass-A column block is
//     16 N2 contiguous words.
// In natural order the rows of a column block are a power of two apart (2 KiB
// at N = 2^16): they fall on 2 of the 16 channels of an XCD's L2 (interleaved
// every 256 bytes), and since the XCD of a workgroup follows from its column
// block, on 4 of 16 over all the workgroups of an XCD.
enum NttLoad : uint32_t {
  kLoadU64 = 0,    // inverse: residues in [0, q) as uint64, natural order
  kLoadF64 = 1,    // forward: integers as doubles, |x| < 2^50, blocked
  kLoadU64T = 2,   // inverse: residues in [0, q) as uint64, transposed
};
enum NttStore : uint32_t {
  kStoreU64T = 0,     // the transform, residues in [0, q) as uint64, transposed
  kStoreF64 = 1,      // the transform, centred residues as doubles, blocked
  kStoreRescale = 2,  // (base - transform) * inv mod q, in [0, q) as uint64, natural order
  kStoreF64C = 3,     // the transform, residues in [0, q) as doubles, blocked
};

// One modulus of a pass and its tables.
struct NttSet {
  const double *mid; // pass A: multiply output (n1, k2) by mid[((n1 / 16) N2 + k2) 16 + n1 mod 16]
  const Tw *dft_a;   // pass A's twiddles: forward N2 (from index 1: 2^s + block), inverse N2 / 2
  const Tw *dft_b;   // size-N1 DFT twiddles (N1 / 2)
  const Tw *post;    // inverse pass B: multiply output k2 + N2 k1 by post[k1] (forward: null)
  Tw inv;            // kStoreRescale: the factor applied after the subtraction
  double q, qinv;    // the modulus and fl(1 / q)
};

// A launch covers vectors v = 0 .. gridDim.y - 1, grouped into sets of vps
// consecutive vectors that share one modulus: vector v is number v % vps of
// set v / vps, whose modulus and tables are sets[v / vps].  Its words sit at
//   in   + (v / vps) * in_set_stride   + (v % vps) * in_stride   + n,
// and likewise for out and base; the intermediate of vector v at
// tmp + v * tmp_words(N1, N2).  Each buffer's end bounds the descriptors of its accesses (buffer_extent).
struct NttPass {
  const void *in;        // pass A input
  double *tmp;           // the transposed intermediates
  void *out;             // pass B output
  const uint64_t *base;  // kStoreRescale: residues in [0, q)
  const NttSet *sets;    // device array, one entry per set
  const uint64_t *add;   // ntt_pass_b_rot: residues in [0, q) added to the first polynomials
  const void *in_end, *tmp_end, *out_end, *base_end, *add_end;   // ends of the buffers above
  uint64_t in_stride, out_stride, base_stride;
  uint64_t in_set_stride, out_set_stride, base_set_stride, add_set_stride;
  uint32_t vps, log_n1, log_n2, load, store;
  uint32_t nt;             // the kernels' NT
  uint32_t nsets_shared;   // pass A: 0, or the number of sets when they all read the same input
                           // vectors (in_set_stride 0) and gridDim.x * vps is a multiple of 8
};

// The passes' global accesses.  These helpers give the work split and the
// byte offsets of every buffer access (VGPR part v, SGPR part s); the
// kernels address memory only through them, and the host replay of a
// launch (ntt_check.hip) runs the same helpers over every workgroup and
// thread to check each access against the buffer it falls in.
struct Off {
  uint32_t v, s;
};

// The intermediate: row k2 is N1 words at k2 (N1 + 16).  The 16 words (128
// bytes) between rows put the rows that one pass-A workgroup writes, 16 words
// of each, on all the L2 channels in turn.
__host__ __device__ constexpr uint32_t tmp_pitch(uint32_t N1) { return N1 + 16; }
__host__ __device__ constexpr size_t tmp_words(uint32_t N1, uint32_t N2) { return (size_t)tmp_pitch(N1) * N2; }

// Pass A over DFT side N2 = 2^LOGM (other side N1): the unit of workgroup
// (bx, by) of a grid gx workgroups wide.
// (With one set per vector, the column blocks go round the XCDs from vector to
// vector, see spread_block.)
struct UnitA {
  uint32_t set, lv, cb;
};
// The block of workgroup (bx, by) of a grid gx (a power of two) wide whose
// blocks are runs of 16 words of the rows of a natural-order vector.  An XCD
// takes every eighth workgroup, so block = bx would keep it on two blocks of
// 16, whose rows share a few L2 channels; this gives it all blocks in turn
// (with the padded intermediate, pass B of 128 ciphertexts' rescale at
// N = 2^16, L = 8: 575 -> 514 us).
__host__ __device__ constexpr uint32_t spread_block(uint32_t bx, uint32_t by, uint32_t gx) {
  return (bx + by) & (gx - 1);
}
__host__ __device__ inline UnitA pass_a_unit(uint32_t vps, uint32_t nsets_shared, uint32_t bx, uint32_t by,
                                             uint32_t gx) {
  UnitA a;
  a.set = by / vps;
  a.lv = by - a.set * vps;
  a.cb = spread_block(bx, by, gx);
  if (nsets_shared) {
    // The sets read the same input vectors: give the nsets_shared workgroups
    // of one (vector, column block) consecutive turns on one XCD (workgroup
    // ids i, i + 8, ... run there), so that the input is fetched once into
    // its L2.  The launch covers gx * vps units, a multiple of 8.
    const uint32_t id = by * gx + bx;
    const uint32_t u = id >> 3, unit = (id & 7u) + 8u * (u / nsets_shared);
    a.set = u % nsets_shared;
    a.lv = unit / gx;
    a.cb = unit - a.lv * gx;
  }
  return a;
}

// Pass B's vector of workgroup row by of a grid of nv rows: all sets of a local
// vector in turn, the order in which pass A with shared inputs writes them.
struct UnitB {
  uint32_t set, lv;
};
__host__ __device__ inline UnitB pass_b_unit(uint32_t vps, uint32_t nv, uint32_t by) {
  const uint32_t nsets = nv / vps, lv = by / nsets;
  return UnitB{by - lv * nsets, lv};
}

template <uint32_t LOGM>
struct GeomA {
  using D = DftShape<LOGM>;
  // first groups, loop index it < IT1: column and group (kLoadU64T walks a column's groups first)
  static __host__ __device__ uint32_t col(uint32_t it, bool trans) { return trans ? it / D::I1 : it % kNttCols; }
  static __host__ __device__ uint32_t grp(uint32_t it, bool trans) { return trans ? it % D::I1 : it / kNttCols; }
  // word u of the first group ip of column n1 (row n2 = ip + I1 rev4(u))
  static __host__ __device__ Off in(uint32_t n1, uint32_t ip, uint32_t u, uint32_t N1) {
    return Off{(n1 + N1 * ip) * 8, N1 * D::I1 * 8 * rev4(u)};
  }
  // the same element in the transposed layout: n = n1 + N1 n2 at (n mod N2) N1 + n / N2
  static __host__ __device__ Off in_t(uint32_t n1, uint32_t ip, uint32_t u, uint32_t N1) {
    const uint32_t n = n1 + N1 * (ip + D::I1 * rev4(u));
    return Off{((n & (D::M - 1)) * N1 + (n >> LOGM)) * 8, 0};
  }
  // the same element in the blocked layout: column cl of block cb
  // (word v is row ip + I1 v)
  static __host__ __device__ Off in_b(uint32_t cb, uint32_t cl, uint32_t ip, uint32_t v) {
    return Off{((cb * D::M + ip) * kNttCols + cl) * 8, D::I1 * kNttCols * 8 * v};
  }
  // last groups, loop index it < IT2: column, offset; word u is row k2 = o + (u << S0L)
  static __host__ __device__ uint32_t col2(uint32_t it) { return it % kNttCols; }
  static __host__ __device__ uint32_t off2(uint32_t it) { return it / kNttCols; }
  static __host__ __device__ Off tmp(uint32_t o, uint32_t n1, uint32_t u, uint32_t N1) {
    return Off{(o * tmp_pitch(N1) + n1) * 8, ((u << D::S0L) * tmp_pitch(N1)) * 8};
  }
  static __host__ __device__ Off mid(uint32_t cb, uint32_t cl, uint32_t o, uint32_t u) {
    return Off{((cb * D::M + o) * kNttCols + cl) * 8, (u << D::S0L) * kNttCols * 8};
  }
};

// Pass B over DFT side N1 = 2^LOGM (other side N2), workgroup rows r0 .. r0 + 15.
template <uint32_t LOGM>
struct GeomB {
  using D = DftShape<LOGM>;
  // first groups, it < IT1: row of the workgroup and group; word u from the row's start
  static __host__ __device__ uint32_t row(uint32_t it) { return it / D::I1; }
  static __host__ __device__ uint32_t grp(uint32_t it) { return it % D::I1; }
  static __host__ __device__ Off tmp(uint32_t row, uint32_t ip, uint32_t u) {
    return Off{(row * tmp_pitch(D::M) + ip) * 8, D::I1 * 8 * rev4(u)};
  }
  // last groups, it < IT2: row and offset (kStoreU64T walks a row's offsets first)
  static __host__ __device__ uint32_t row2(uint32_t it, bool trans) { return trans ? it / D::I2 : it % kNttCols; }
  static __host__ __device__ uint32_t off2(uint32_t it, bool trans) { return trans ? it % D::I2 : it / kNttCols; }
  static __host__ __device__ Off post(uint32_t o, uint32_t u) { return Off{o * 16, (u << D::S0L) * 16}; }
  // output k2 + N2 k1, k1 = o + (u << S0L), in natural order, transposed and blocked
  static __host__ __device__ Off col(uint32_t k2, uint32_t o, uint32_t u, uint32_t N2) {
    return Off{(k2 + N2 * o) * 8, (N2 * 8 << D::S0L) * u};
  }
  static __host__ __device__ Off row_t(uint32_t k2, uint32_t o, uint32_t u) {
    return Off{(k2 * D::M + o) * 8, (u << D::S0L) * 8};
  }
  // (N1 = N2 2^d, d = 0 or 1: n1 = k2 + N2 (k1 mod 2^d), n2 = k1 >> d)
  static __host__ __device__ Off block(uint32_t k2, uint32_t o, uint32_t u, uint32_t N2) {
    const uint32_t d = D::M / N2 - 1, b = k2 / kNttCols + (N2 / kNttCols) * (o & d);
    return Off{((b * N2 + (o >> d)) * kNttCols + k2 % kNttCols) * 8, ((u << D::S0L) >> d) * kNttCols * 8};
  }
};

// The fused pass B of the rotations (ntt_pass_b_rot, rotate.hip) over DFT
// side N1 = 2^LOGM: destination columns d_lo = o0 .. o0 + 15 of the rotation
// by Galois element g.
constexpr uint32_t kRotMax = 256;   // rotations per call (their Galois elements ride in the arguments)

struct RotArgs {
  uint32_t g[kRotMax];
  uint32_t n_rot, L;
  uint32_t lv0;          // the launch's vectors are numbers lv0, lv0 + 1, ... of the 2 n_rot
  uint32_t c0_natural;   // NttPass::add is in natural order, not transposed
};

template <uint32_t LOGM>
struct GeomRot {
  using D = DftShape<LOGM>;
  static constexpr uint32_t PER = kNttCols * D::M / kNttThreads;   // stores per thread
  // first groups, it < IT1: the workgroup's column and group
  static __host__ __device__ uint32_t row(uint32_t it) { return it / D::I1; }
  static __host__ __device__ uint32_t grp(uint32_t it) { return it % D::I1; }
  // the intermediate row k2 that destination column d_lo reads
  static __host__ __device__ uint32_t src_row(uint32_t g, uint32_t d_lo, uint32_t N2) {
    return (g * d_lo + (g - 1) / 2) & (N2 - 1);
  }
  static __host__ __device__ Off tmp(uint32_t k2, uint32_t ip, uint32_t u) {
    return Off{(k2 * tmp_pitch(D::M) + ip) * 8, D::I1 * 8 * rev4(u)};
  }
  // last groups, it < IT2: the workgroup's column and offset; word k1 = o + (u << S0L) of row k2
  static __host__ __device__ uint32_t row2(uint32_t it) { return it / D::I2; }
  static __host__ __device__ uint32_t off2(uint32_t it) { return it % D::I2; }
  static __host__ __device__ Off word(uint32_t k2, uint32_t o, uint32_t u) {
    return Off{(k2 * D::M + o) * 8, (u << D::S0L) * 8};
  }
  // the same word in natural order
  static __host__ __device__ Off natural(uint32_t k2, uint32_t o, uint32_t u, uint32_t N2) {
    return Off{(k2 + N2 * o) * 8, (N2 * 8 << D::S0L) * u};
  }
  // store j of thread t: column o0 + t mod 16, destination row d_hi = t / 16 + 16 j
  static __host__ __device__ Off out(uint32_t o0, uint32_t t, uint32_t j, uint32_t N2) {
    return Off{(o0 + t % kNttCols + (t / kNttCols) * N2) * 8, j * kNttCols * N2 * 8};
  }
};

// Pass A, N2 = 2^LOGM: grid (N1 / kNttCols, vectors).  The first groups of
// column n1 hold rows n2 = i' + I1 v; the quarter waves read runs of
// kNttCols columns of one row (kLoadU64T: runs of consecutive rows of one
// column, which are contiguous there).  FWD: the forward transform (kLoadF64).
// NT: nontemporal stores; a kernel of its own, as both policies' stores in one
// cost the smallest calls 0.1 us a launch.
// What bounds it: the L1 path (it serves one 64-byte access a clock), the
// arithmetic and the stores take about the same time and overlap badly
// (parts taken out one at a time, N = 2^16, L = 8, 128 ciphertexts, of 444 us:
// stores 160, loads 113, mid 57, a separate twist 36; arithmetic alone 221).
// So the twist rides in the butterflies (no loads, no products) and mid is one
// double a word instead of a twiddle pair: 447 -> 393 us.  The input is issued
// before the set record and the twiddles are read, and mid (pass B: the
// minuends) before the barrier, so that their latencies overlap: the whole
// rescale 980 -> 932 us (loads that pass B issued ahead of its input instead
// cost 1%: they return in order).  The last groups store rows
// k2 = o + (u << S0L) of the intermediate, again in runs of kNttCols columns.
template <uint32_t LOGM, bool FWD, bool NT>
__global__ void __launch_bounds__(kNttThreads) ntt_pass_a(const NttPass P) {
  static_assert(dft_out<LOGM>() < 4, "mid's input");
  using D = DftShape<LOGM>;
  using G = GeomA<LOGM>;
  extern __shared__ double xs[];   // [kNttCols][PM], then the transform's twiddles
  Tw *tw = (Tw *)(xs + kNttCols * D::PM);
  const UnitA un = pass_a_unit(P.vps, P.nsets_shared, blockIdx.x, blockIdx.y, gridDim.x);
  const uint32_t set = un.set, lv = un.lv, cb = un.cb;
  const uint32_t log_n1 = P.log_n1, N1 = 1u << log_n1, N2 = D::M;
  const uint64_t v = (uint64_t)set * P.vps + lv;
  const uint64_t in_off = set * P.in_set_stride + lv * P.in_stride;
  const bool trans = P.load == kLoadU64T;   // uniform
  const Buf in((const char *)P.in + in_off * 8, P.in_end);
  uint64_t w[16];   // the words of a first group, as loaded
  auto load = [&](uint32_t it) {
    const uint32_t cl = G::col(it, trans), ip = G::grp(it, trans), n1 = cb * kNttCols + cl;
    if (!FWD && !trans) {
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) {
        const Off o = G::in(n1, ip, u, N1);
        w[u] = in.u64(o.v, o.s);
      }
    } else {
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) {
        const Off o = FWD ? G::in_b(cb, cl, ip, u) : G::in_t(n1, ip, u, N1);
        w[u] = in.u64(o.v, o.s);
      }
    }
  };
  if (threadIdx.x < D::IT1) load(threadIdx.x);   // in flight while the set record and the twiddles arrive
  const NttSet S = P.sets[set];
  stage_twiddles(tw, S.dft_a, FWD ? D::M : D::M / 2);
  Tw t1[8];
  if constexpr (!FWD) first_twiddles<LOGM>(t1, S.dft_a);
  const double q = S.q, qinv = S.qinv;
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < D::IT1; it += kNttThreads) {
    const uint32_t cl = G::col(it, trans), ip = G::grp(it, trans);
    if (D::IT1 > kNttThreads && it != threadIdx.x) load(it);
    double r[16];
    if constexpr (FWD) {
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) r[u] = __builtin_bit_cast(double, w[u]);
      tree_first<LOGM>(xs, cl, ip, r, S.dft_a, q, qinv);
    } else {
#pragma unroll
      for (uint32_t u = 0; u < 16; ++u) r[u] = to_f64(w[u]);
      first_stages<LOGM>(r, t1, q, qinv);
      put_first<LOGM>(xs, cl, ip, r, q, qinv);
    }
  }
  const Buf tmp(P.tmp + v * tmp_words(N1, N2), P.tmp_end), mid(S.mid, S.mid + (size_t)N1 * N2);
  double m[D::E2];   // mid of a last group
  auto load_mid = [&](uint32_t it) {
#pragma unroll
    for (uint32_t u = 0; u < D::E2; ++u) {
      const Off om = G::mid(cb, G::col2(it), G::off2(it), u);
      m[u] = mid.f64(om.v, om.s);
    }
  };
  load_mid(threadIdx.x);   // in flight over the barrier and the last stages
  static_assert(D::S0L == 4, "the last groups follow the first");
  __syncthreads();
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < D::IT2; it += kNttThreads) {
    const uint32_t cl = G::col2(it), o = G::off2(it), n1 = cb * kNttCols + cl;
    if (D::IT2 > kNttThreads && it != threadIdx.x) load_mid(it);
    double r[D::E2];
    if constexpr (FWD) tree_last<LOGM>(xs, cl, o, tw, r, q);
    else last_stages<LOGM>(xs, cl, o, tw, r, q, qinv);
#pragma unroll
    for (uint32_t u = 0; u < D::E2; ++u) {
      const Off ot = G::tmp(o, n1, u, N1);
      const uint32_t e = FWD ? rev4(u) >> (4 - D::R2) : u;
      tmp.put<NT>(mul_tw(r[e], Tw{m[u], m[u] * qinv}, q), ot.v, ot.s);
    }
  }
}

// Pass B, N1 = 2^LOGM: grid (N2 / kNttCols, vectors).  The first groups read
// runs of I1 consecutive words of one intermediate row k2; the last groups
// store column k2 = r0 + (lane mod kNttCols), rows k1, as runs of kNttCols
// words (kStoreU64T: runs of consecutive k1 of one row k2; blocked: rows k1
// and k1 + 2^d follow each other).  INV: the inverse transform (post, centred or
// residues as doubles), else the forward one (to residues, kStoreRescale or
// kStoreU64T).  Two kernels: in a common one the minuends held over the barrier
// left the compiler no registers for post, and its 16 loads waited one for
// another (inverse passes B of 4 / 12 ciphertexts' rescales at L = 3 17.6 us at
// N = 2^17 and 8.7 at 2^15, before the minuends were moved 12.2 and 7.7).  With
// post ahead of the barrier as well, rescales in us, common -> two kernels:
// N = 2^17, L = 3, 4 ciphertexts 52.0 -> 45.1; 2^16, L = 6, 4 42.2 -> 39.2,
// L = 16, 4 67.4 -> 64.0; 2^15, L = 3, 12 37.1 -> 34.4.
template <uint32_t LOGM, bool INV, bool NT>
__global__ void __launch_bounds__(kNttThreads) ntt_pass_b(const NttPass P) {
  using D = DftShape<LOGM>;
  using G = GeomB<LOGM>;
  extern __shared__ double xs[];   // [kNttCols][PM], then the M/2 DFT twiddles
  Tw *tw = (Tw *)(xs + kNttCols * D::PM);
  const UnitB un = pass_b_unit(P.vps, gridDim.y, blockIdx.y);
  const uint32_t set = un.set, lv = un.lv;
  const uint32_t N2 = 1u << P.log_n2, M = D::M;
  const uint32_t r0 = spread_block(blockIdx.x, blockIdx.y, gridDim.x) * kNttCols;
  const uint64_t v = (uint64_t)set * P.vps + lv;
  const Buf tmp(P.tmp + v * tmp_words(M, N2) + (size_t)r0 * tmp_pitch(M), P.tmp_end);
  double x[16];   // a first group, as loaded
  auto load = [&](uint32_t it) {
#pragma unroll
    for (uint32_t u = 0; u < 16; ++u) {
      const Off o = G::tmp(G::row(it), G::grp(it), u);
      x[u] = tmp.f64_once(o.v, o.s);
    }
  };
  if (threadIdx.x < D::IT1) load(threadIdx.x);   // in flight while the set record and the twiddles arrive
  const NttSet S = P.sets[set];
  stage_twiddles(tw, S.dft_b, D::M / 2);
  Tw t1[8];
  first_twiddles<LOGM>(t1, S.dft_b);
  const double q = S.q, qinv = S.qinv;
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < D::IT1; it += kNttThreads) {
    if (D::IT1 > kNttThreads && it != threadIdx.x) load(it);
    first_stages<LOGM>(x, t1, q, qinv);
    put_first<LOGM>(xs, G::row(it), G::grp(it), x, q, qinv);
  }
  const bool transposed = !INV && P.store == kStoreU64T, rescale = !INV && !transposed;   // uniform
  const Buf out((const char *)P.out + (set * P.out_set_stride + lv * P.out_stride) * 8, P.out_end);
  const Buf base(rescale ? P.base + set * P.base_set_stride + lv * P.base_stride : nullptr,
                 rescale ? P.base_end : nullptr);
  uint64_t bv[D::E2];   // the minuends of a last group
  auto load_base = [&](uint32_t it) {
#pragma unroll
    for (uint32_t u = 0; u < D::E2; ++u) {
      const Off oc = G::col(r0 + G::row2(it, false), G::off2(it, false), u, N2);
      bv[u] = base.u64_once(oc.v, oc.s);
    }
  };
  const Buf post(S.post, INV ? S.post + M : S.post);
  double pw[D::E2];   // post of a last group (w only, half the registers of the pair; w / q as w fl(1/q), like mid's)
  auto load_post = [&](uint32_t it) {
#pragma unroll
    for (uint32_t u = 0; u < D::E2; ++u) {
      const Off op = G::post(G::off2(it, false), u);
      pw[u] = post.f64(op.v, op.s);
    }
  };
  // in flight over the barrier and the last stages
  if constexpr (INV) load_post(threadIdx.x);
  else if (rescale) load_base(threadIdx.x);
  middle_stages<LOGM>(xs, tw, q, qinv);
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < D::IT2; it += kNttThreads) {
    const uint32_t row = G::row2(it, transposed), o = G::off2(it, transposed);
    const uint32_t k2 = r0 + row;   // output k2 + N2 k1, k1 = o + (u << S0L)
    if (D::IT2 > kNttThreads && it != threadIdx.x) {
      if constexpr (INV) load_post(it);
      else if (rescale) load_base(it);
    }
    double y[D::E2];
    last_stages<LOGM>(xs, row, o, tw, y, q, qinv);
    if constexpr (INV) {
#pragma unroll
      for (uint32_t u = 0; u < D::E2; ++u) y[u] = mul_tw(y[u], Tw{pw[u], pw[u] * qinv}, q);
#pragma unroll
      for (uint32_t u = 0; u < D::E2; ++u) {
        const Off ob = G::block(k2, o, u, N2);
        double z = reduce(y[u], q, qinv);
        if (P.store == kStoreF64C && z < 0.0) z += q;
        out.put<NT>(z, ob.v, ob.s);
      }
    } else if (rescale) {
#pragma unroll
      for (uint32_t u = 0; u < D::E2; ++u) {
        const Off oc = G::col(k2, o, u, N2);
        const double z = mul_tw(minuend<reduce_minuend<LOGM>()>(bv[u], y[u], q, qinv), S.inv, q);
        out.put(to_u64(canonical(z, q, qinv)), oc.v, oc.s);
      }
    } else {
#pragma unroll
      for (uint32_t u = 0; u < D::E2; ++u) {
        const Off ot = G::row_t(k2, o, u);
        out.put(to_u64(canonical(y[u], q, qinv)), ot.v, ot.s);
      }
    }
  }
}

}  // namespace fiona
