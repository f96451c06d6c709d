// Whole transforms in one workgroup, for rings whose vector of N doubles fits
// the LDS next to its padding and twiddles (N <= 2^14): the rescale and the
// rotations' digits and division by P, each as one launch.
//
// What bounds the passes of ntt_kernel.hpp at these sizes is their number: a
// launch costs the host 3.3 us and the GPU 4 to 5 us however small it is, and
// at larger counts their intermediates and the half of their threads that a
// side of 128 leaves idle.  Measured when the passes went there too, passes ->
// one launch: rescale at L = 6 of 4 / 128 ciphertexts, N = 2^10 17.0 -> 6.9 /
// 30.2 -> 14.6 us, 2^12 17.2 -> 9.9 / 66.3 -> 32.8, 2^13 17.6 -> 15.7 / 104 -> 58;
// rotations at L = 6, 4 / 64 of them, N = 2^11 43.0 -> 24.2 / 81.3 -> 64.2, 2^12
// 43.1 -> 31.3 / 102 -> 82.
//
// The four-step transform of ntt_kernel.hpp with its intermediate in LDS: the
// N1 columns of N2 words lie padded_len(N2) apart, and every step works in
// place, so that no word leaves the CU between the first load and the last
// store.  A workgroup transforms one vector back to its coefficients, keeps
// them in registers (4, 8 or 16 a thread), and transforms them forward under the
// moduli of its group, one after the other.  Splitting the moduli over several
// groups repeats the inverse transform in each, which a small call pays for
// idle CUs (whole_groups).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "buffer.hpp"
#include "ntt_kernel.hpp"

namespace fiona {

// A transform of side 2^LOGM in two groups of stages, R1 then R2: 2 + 2, 3 + 2,
// 3 + 3 or 4 + 3.  Short groups and many threads: a call of few vectors waits
// for one thread's chain of instructions.  With groups of 16 words at every
// size, the rescale of 4 ciphertexts at L = 3 took 11.6 us at N = 2^10 and
// 2^11, 12.4 at 2^12 and 17.3 at 2^13; with these 6.9, 7.3, 9.8 and 15.4.
template <uint32_t LOGM>
struct Side {
  static constexpr uint32_t M = 1u << LOGM, R1 = LOGM == 4 ? 2 : LOGM == 7 ? 4 : 3, R2 = LOGM - R1;
  static constexpr uint32_t E1 = 1u << R1, E2 = 1u << R2;   // words of a first and a last group
  static_assert(LOGM >= 4 && LOGM <= 7 && R1 <= 4 && R2 <= 4, "groups of up to 16 words");
  static constexpr double kOut = transform_out<LOGM, R1>();   // the outputs' bound
  static __host__ __device__ constexpr uint32_t rev1(uint32_t u) { return rev4(u) >> (4 - R1); }
  static __host__ __device__ constexpr uint32_t rev2(uint32_t u) { return rev4(u) >> (4 - R2); }
};

template <uint32_t LN>
struct Whole {
  static constexpr uint32_t LOG1 = (LN + 1) / 2, LOG2 = LN / 2, N = 1u << LN, N1 = 1u << LOG1, N2 = 1u << LOG2;
  using A = Side<LOG2>;
  using B = Side<LOG1>;
  static constexpr uint32_t T = N / A::E1;                      // threads: one first group of pass A each
  static constexpr uint32_t PM = padded_len(N2), WORDS = N1 * PM;   // LDS words of a column and of the vector
};

// The kernels' indexes: LDS words, and byte offsets from each buffer's base.
// They address memory and LDS only through these, and the host replay of a
// launch (ntt_check.hip) runs them over every workgroup and thread.
template <uint32_t LN>
struct GeomWhole {
  using W = Whole<LN>;
  using A = typename W::A;
  using B = typename W::B;
  static constexpr uint32_t N = W::N, N1 = W::N1, N2 = W::N2;
  // the LDS word of row position p, column c
  static __host__ __device__ constexpr uint32_t at(uint32_t p, uint32_t c) { return c * W::PM + pidx(p); }
  // the column that holds output k1 = o + E1 u of a row (pass B works in place:
  // first group i' leaves word u of its results in column i' + E2 u)
  static __host__ __device__ constexpr uint32_t col(uint32_t o, uint32_t u) { return B::rev2(u) + B::E2 * o; }
  // pass A's first groups: thread t's column n1 and group i'
  static __host__ __device__ constexpr uint32_t col1(uint32_t t) { return t % N1; }
  static __host__ __device__ constexpr uint32_t grp1(uint32_t t) { return t / N1; }
  // word u of the inverse's group (element coef(n1, i', rev1(u))), and where result u goes
  static __host__ __device__ constexpr uint32_t coef(uint32_t n1, uint32_t ip, uint32_t v) {
    return n1 + N1 * (ip + A::E2 * v);
  }
  static __host__ __device__ constexpr uint32_t in(uint32_t n1, uint32_t ip, uint32_t u, bool trans) {
    const uint32_t n = coef(n1, ip, A::rev1(u));
    return (trans ? (n % N2) * N1 + n / N2 : n) * 8;
  }
  // (inverse: i = rev2(i'))
  static __host__ __device__ constexpr uint32_t first_inv(uint32_t n1, uint32_t i, uint32_t u) {
    return at(A::E1 * i + u, n1);
  }
  static __host__ __device__ constexpr uint32_t first_fwd(uint32_t n1, uint32_t ip, uint32_t u) {
    return at(u * A::E2 + ip, n1);
  }
  // pass A's last groups, loop index it < N / A::E2: column, and o of the outputs
  // k2 = o + E1 u (forward: words of block j = rev1(o))
  static constexpr uint32_t IT2 = N / A::E2;
  static __host__ __device__ constexpr uint32_t col2(uint32_t it) { return it % N1; }
  static __host__ __device__ constexpr uint32_t off2(uint32_t it) { return it / N1; }
  static __host__ __device__ constexpr Off mid(uint32_t c, uint32_t o, uint32_t u) {
    return Off{(((c / kNttCols) * N2 + o) * kNttCols + c % kNttCols) * 8, A::E1 * u * kNttCols * 8};
  }
  static __host__ __device__ constexpr uint32_t last_a(uint32_t c, uint32_t o, uint32_t j, uint32_t e, bool fwd) {
    return at(fwd ? j * A::E2 + e : o + A::E1 * e, c);
  }
  // pass B's first groups, it < N / B::E1: row position p and group i'; word u read and written
  static constexpr uint32_t IT3 = N / B::E1;
  static __host__ __device__ constexpr uint32_t pos3(uint32_t it) { return it % N2; }
  static __host__ __device__ constexpr uint32_t grp3(uint32_t it) { return it / N2; }
  static __host__ __device__ constexpr uint32_t b_in(uint32_t p, uint32_t ip, uint32_t u) {
    return at(p, ip + B::E2 * B::rev1(u));
  }
  static __host__ __device__ constexpr uint32_t b_out(uint32_t p, uint32_t ip, uint32_t u) {
    return at(p, ip + B::E2 * u);
  }
  // its last groups, it < N / B::E2: row k2 and o of the outputs k1 = o + E1 u, rows first or (rowwise) a row's o first
  static constexpr uint32_t IT4 = N / B::E2;
  static __host__ __device__ constexpr uint32_t row4(uint32_t it, bool rowwise) { return rowwise ? it / B::E1 : it % N2; }
  static __host__ __device__ constexpr uint32_t off4(uint32_t it, bool rowwise) { return rowwise ? it % B::E1 : it / N2; }
  // the row position of k2 after a forward pass A
  static __host__ __device__ constexpr uint32_t pos_fwd(uint32_t k2) { return bit_reverse(k2, W::LOG2); }
  static __host__ __device__ constexpr uint32_t last_b(uint32_t p, uint32_t o, uint32_t u) { return at(p, col(o, u)); }
  static __host__ __device__ constexpr Off post(uint32_t o, uint32_t u) { return Off{o * 16, u * B::E1 * 16}; }
  // output (k2, k1 = o + E1 u) in natural order and transposed
  static __host__ __device__ constexpr Off natural(uint32_t k2, uint32_t o, uint32_t u) {
    return Off{(k2 + N2 * o) * 8, N2 * B::E1 * 8 * u};
  }
  static __host__ __device__ constexpr Off row(uint32_t k2, uint32_t o, uint32_t u) {
    return Off{(k2 * N1 + o) * 8, u * B::E1 * 8};
  }
  // the LDS word of output k, its row at position p
  static __host__ __device__ constexpr uint32_t word(uint32_t p, uint32_t k) {
    return at(p, col((k / N2) % B::E1, (k / N2) / B::E1));
  }
  // destination d of the automorphism by g takes slot pi(d) = g d + (g - 1) / 2 mod N
  static __host__ __device__ constexpr uint32_t slot(uint32_t g, uint32_t d) { return (g * d + (g - 1) / 2) & (N - 1); }
  static __host__ __device__ constexpr uint32_t dest(uint32_t d) { return d * 8; }
};

// The vector and the moduli [first, last) of n of workgroup b, the moduli in `groups` groups.
struct WholeUnit {
  uint32_t v, first, last;
};
__host__ __device__ inline WholeUnit whole_unit(uint32_t b, uint32_t groups, uint32_t n) {
  const uint32_t v = b / groups, g = b - v * groups;
  return WholeUnit{v, n * g / groups, n * (g + 1) / groups};
}
template <uint32_t LN>
constexpr size_t whole_smem() {
  using W = Whole<LN>;
  return W::WORDS * sizeof(double) + (W::N2 + W::N1 / 2) * sizeof(Tw);
}
static_assert(whole_smem<12>() <= 64 * 1024, "from 2^13 on the kernels are given more LDS than by default");

// The two passes' twiddles of one set into LDS (tw_a, then tw_b).
template <uint32_t LN>
__device__ __forceinline__ void whole_twiddles(Tw *tw_a, Tw *tw_b, const NttSet &S, bool fwd) {
  using W = Whole<LN>;
  for (uint32_t i = threadIdx.x; i < (fwd ? W::N2 : W::N2 / 2); i += W::T) tw_a[i] = S.dft_a[i];
  for (uint32_t i = threadIdx.x; i < W::N1 / 2; i += W::T) tw_b[i] = S.dft_b[i];
}

// The first stages of a cyclic DFT of side 2^LOGM on r[u] = word i' + E2
// rev1(u), twiddles uniform over the workgroup.
template <uint32_t LOGM>
__device__ __forceinline__ void whole_first(double (&r)[Side<LOGM>::E1], const Tw *__restrict__ dft, double q,
                                            double qinv) {
  using D = Side<LOGM>;
  butterflies<LOGM, 0, D::R1>(r, 0, [&](uint32_t t) { return dft[t]; }, q, qinv);
}

// Pass A's last groups, the product with mid, and pass B's first groups, in
// place; barriers before, between and after.  FWD: row position of output k2
// is bitrev(k2), else k2.
template <uint32_t LN, bool FWD>
__device__ __forceinline__ void whole_middle(double *xs, const Tw *tw_a, const NttSet &S) {
  using W = Whole<LN>;
  using A = typename W::A;
  using B = typename W::B;
  using G = GeomWhole<LN>;
  const double q = S.q, qinv = S.qinv;
  const Buf mid(S.mid, S.mid + W::N);
  __syncthreads();
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < G::IT2; it += W::T) {
    const uint32_t c = G::col2(it), o = G::off2(it), j = A::rev1(o);
    double m[A::E2], r[A::E2];
#pragma unroll
    for (uint32_t u = 0; u < A::E2; ++u) {
      const Off om = G::mid(c, o, u);
      m[u] = mid.f64(om.v, om.s);
    }
#pragma unroll
    for (uint32_t e = 0; e < A::E2; ++e) r[e] = xs[G::last_a(c, o, j, e, FWD)];
    if constexpr (FWD) tree_butterflies<A::R1, A::R2>(r, j, [&](uint32_t t) { return tw_a[t]; }, q);
    else butterflies<W::LOG2, A::R1, A::R2>(r, o, [&](uint32_t t) { return tw_a[t]; }, q, qinv);
#pragma unroll
    for (uint32_t e = 0; e < A::E2; ++e) {
      const double w = m[FWD ? A::rev2(e) : e];
      xs[G::last_a(c, o, j, e, FWD)] = mul_tw(r[e], Tw{w, w * qinv}, q);
    }
  }
  __syncthreads();
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < G::IT3; it += W::T) {
    const uint32_t p = G::pos3(it), ip = G::grp3(it);
    double r[B::E1];
#pragma unroll
    for (uint32_t u = 0; u < B::E1; ++u) r[u] = xs[G::b_in(p, ip, u)];
    whole_first<W::LOG1>(r, S.dft_b, q, qinv);
#pragma unroll
    for (uint32_t u = 0; u < B::E1; ++u) xs[G::b_out(p, ip, u)] = reduce(r[u], q, qinv);
  }
  __syncthreads();
}

// Pass B's last groups: y[u] is output (k2, k1 = o + E1 u), its row at position p.
template <uint32_t LN>
__device__ __forceinline__ void whole_last(const double *xs, uint32_t p, uint32_t o, const Tw *tw_b,
                                           double (&y)[Whole<LN>::B::E2], const NttSet &S) {
  using W = Whole<LN>;
#pragma unroll
  for (uint32_t u = 0; u < W::B::E2; ++u) y[u] = xs[GeomWhole<LN>::last_b(p, o, u)];
  butterflies<W::LOG1, W::B::R1, W::B::R2>(y, o, [&](uint32_t t) { return tw_b[t]; }, S.q, S.qinv);
}

// The inverse transform of the vector at `in` (residues as uint64; TRANS: in
// the transposed layout): on return w[v] is coefficient n1 + N1 (i' + E2 v) of
// thread (n1 = tid mod N1, i' = tid / N1), the centred residue, or with CANON
// the one in [0, q).
template <uint32_t LN, bool TRANS, bool CANON>
__device__ __forceinline__ void whole_inverse(double *xs, Tw *tw_a, Tw *tw_b, const Buf &in, const NttSet *sets,
                                              double (&w)[Whole<LN>::A::E1]) {
  using W = Whole<LN>;
  using A = typename W::A;
  using B = typename W::B;
  using G = GeomWhole<LN>;
  const uint32_t n1 = G::col1(threadIdx.x), ip = G::grp1(threadIdx.x);
  uint64_t x[A::E1];
#pragma unroll
  for (uint32_t u = 0; u < A::E1; ++u) x[u] = in.u64(G::in(n1, ip, u, TRANS), 0);
  const NttSet S = *sets;
  const double q = S.q, qinv = S.qinv;
  whole_twiddles<LN>(tw_a, tw_b, S, false);
  {
    double r[A::E1];
#pragma unroll
    for (uint32_t u = 0; u < A::E1; ++u) r[u] = to_f64(x[u]);
    whole_first<W::LOG2>(r, S.dft_a, q, qinv);
    const uint32_t i = A::rev2(ip);
#pragma unroll
    for (uint32_t u = 0; u < A::E1; ++u) xs[G::first_inv(n1, i, u)] = reduce(r[u], q, qinv);
  }
  whole_middle<LN, false>(xs, tw_a, S);
  const Buf post(S.post, S.post + W::N1);
#pragma unroll 1
  for (uint32_t it = threadIdx.x; it < G::IT4; it += W::T) {
    const uint32_t k2 = G::row4(it, false), o = G::off4(it, false);
    double y[B::E2];
    whole_last<LN>(xs, k2, o, tw_b, y, S);
#pragma unroll
    for (uint32_t u = 0; u < B::E2; ++u) {
      const Off op = G::post(o, u);
      double z = reduce(mul_tw(y[u], post.tw(op.v, op.s), q), q, qinv);
      if (CANON && z < 0.0) z += q;
      xs[G::last_b(k2, o, u)] = z;
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t v = 0; v < A::E1; ++v) {
    const uint32_t n = G::coef(n1, ip, v);
    w[v] = xs[G::word(n % W::N2, n)];
  }
  __syncthreads();
}

// The forward transform of w (as whole_inverse leaves it) up to pass B's last
// groups.  The caller has a barrier between its last LDS access and this.
template <uint32_t LN>
__device__ __forceinline__ void whole_forward(double *xs, Tw *tw_a, Tw *tw_b, const double (&w)[Whole<LN>::A::E1],
                                              const NttSet &S) {
  using W = Whole<LN>;
  using A = typename W::A;
  using G = GeomWhole<LN>;
  whole_twiddles<LN>(tw_a, tw_b, S, true);
  const uint32_t n1 = G::col1(threadIdx.x), ip = G::grp1(threadIdx.x);
  double r[A::E1];
#pragma unroll
  for (uint32_t v = 0; v < A::E1; ++v) r[v] = w[v];
  const Tw *__restrict__ tree = S.dft_a;
  tree_butterflies<0, A::R1>(r, 0, [&](uint32_t t) { return tree[t]; }, S.q);
#pragma unroll
  for (uint32_t v = 0; v < A::E1; ++v) xs[G::first_fwd(n1, ip, v)] = reduce(r[v], S.q, S.qinv);
  whole_middle<LN, true>(xs, tw_a, S);
}

// (four waves per SIMD: 1,024 threads are as many.  It leaves 128 registers, and
// whole_divide_kernel<13> spills five words a thread.)
#define FIONA_WHOLE_KERNEL(LN) \
  __global__ void __launch_bounds__(Whole<LN>::T) __attribute__((amdgpu_waves_per_eu(4)))

// One rescale: workgroup = (vector v of the 2 n_ct, group g of the L - 1 limbs);
// sets as the rescaler's (forward limbs, then the last limb's inverse).
template <uint32_t LN>
FIONA_WHOLE_KERNEL(LN)
whole_rescale_kernel(const uint64_t *in, uint64_t *out, const NttSet *sets, uint32_t L, uint32_t groups,
                     const void *in_end, const void *out_end) {
  using W = Whole<LN>;
  extern __shared__ double xs[];
  Tw *tw_a = (Tw *)(xs + W::WORDS), *tw_b = tw_a + W::N2;
  using G = GeomWhole<LN>;
  const WholeUnit un = whole_unit(blockIdx.x, groups, L - 1);
  const uint32_t v = un.v;
  double w[W::A::E1];
  whole_inverse<LN, false, false>(xs, tw_a, tw_b, Buf(in + ((size_t)v * L + L - 1) * W::N, in_end), sets + (L - 1), w);
#pragma unroll 1
  for (uint32_t l = un.first; l < un.last; ++l) {
    const NttSet S = sets[l];
    const double q = S.q, qinv = S.qinv;
    const Buf base(in + ((size_t)v * L + l) * W::N, in_end), o_buf(out + ((size_t)v * (L - 1) + l) * W::N, out_end);
    whole_forward<LN>(xs, tw_a, tw_b, w, S);
#pragma unroll 1
    for (uint32_t it = threadIdx.x; it < G::IT4; it += W::T) {
      const uint32_t k2 = G::row4(it, false), o = G::off4(it, false);
      uint64_t b[W::B::E2];
#pragma unroll
      for (uint32_t u = 0; u < W::B::E2; ++u) {
        const Off on = G::natural(k2, o, u);
        b[u] = base.u64_once(on.v, on.s);
      }
      double y[W::B::E2];
      whole_last<LN>(xs, G::pos_fwd(k2), o, tw_b, y, S);
#pragma unroll
      for (uint32_t u = 0; u < W::B::E2; ++u) {
        const Off on = G::natural(k2, o, u);
        const double z = mul_tw(minuend<(W::B::kOut + 1 >= 4)>(b[u], y[u], q, qinv), S.inv, q);
        o_buf.put(to_u64(canonical(z, q, qinv)), on.v, on.s);
      }
    }
    if (l + 1 < un.last) __syncthreads();   // uniform over the workgroup
  }
}

// The rotations' digits: workgroup = (digit j, group g of the L + 1 moduli):
// D_j = INTT(c1_j) in [0, q_j), then Dhat[j][m] = NTT_m(D_j), transposed.
template <uint32_t LN>
FIONA_WHOLE_KERNEL(LN)
whole_digits_kernel(const uint64_t *c1, uint64_t *dhat, const NttSet *inv_sets, const NttSet *fwd_sets, uint32_t L,
                    uint32_t groups, const void *c1_end, const void *dhat_end) {
  using W = Whole<LN>;
  extern __shared__ double xs[];
  Tw *tw_a = (Tw *)(xs + W::WORDS), *tw_b = tw_a + W::N2;
  using G = GeomWhole<LN>;
  const uint32_t M = L + 1;
  const WholeUnit un = whole_unit(blockIdx.x, groups, M);
  const uint32_t j = un.v;
  double w[W::A::E1];
  whole_inverse<LN, false, true>(xs, tw_a, tw_b, Buf(c1 + (size_t)j * W::N, c1_end), inv_sets + j, w);
#pragma unroll 1
  for (uint32_t m = un.first; m < un.last; ++m) {
    const NttSet S = fwd_sets[m];
    const Buf o_buf(dhat + ((size_t)j * M + m) * W::N, dhat_end);
    whole_forward<LN>(xs, tw_a, tw_b, w, S);
#pragma unroll 1
    for (uint32_t it = threadIdx.x; it < G::IT4; it += W::T) {
      const uint32_t k2 = G::row4(it, true), o = G::off4(it, true);
      double y[W::B::E2];
      whole_last<LN>(xs, G::pos_fwd(k2), o, tw_b, y, S);
#pragma unroll
      for (uint32_t u = 0; u < W::B::E2; ++u) {
        const Off ot = G::row(k2, o, u);
        o_buf.put(to_u64(canonical(y[u], S.q, S.qinv)), ot.v, ot.s);
      }
    }
    if (m + 1 < un.last) __syncthreads();
  }
}

// The rotations' division by P and the automorphism: workgroup = (vector lv =
// p n_rot + r, group g of the L limbs); u: [2][n_rot][L + 1][N] transposed, c0
// in natural order, out [n_rot][2][L][N].
template <uint32_t LN>
FIONA_WHOLE_KERNEL(LN)
whole_divide_kernel(const uint64_t *u_in, const uint64_t *c0, uint64_t *out, const NttSet *p_inv_set,
                    const NttSet *down_sets, uint32_t groups, const void *u_end, const void *c0_end,
                    const void *out_end, const RotArgs R) {
  using W = Whole<LN>;
  extern __shared__ double xs[];
  Tw *tw_a = (Tw *)(xs + W::WORDS), *tw_b = tw_a + W::N2;
  using G = GeomWhole<LN>;
  const uint32_t L = R.L, M = L + 1;
  const WholeUnit un = whole_unit(blockIdx.x, groups, L);
  const uint32_t lv = un.v, p = lv / R.n_rot, r = lv - p * R.n_rot, gal = R.g[r];
  double w[W::A::E1];
  whole_inverse<LN, true, false>(xs, tw_a, tw_b, Buf(u_in + ((size_t)lv * M + L) * W::N, u_end), p_inv_set, w);
#pragma unroll 1
  for (uint32_t l = un.first; l < un.last; ++l) {
    const NttSet S = down_sets[l];
    const double q = S.q, qinv = S.qinv;
    const Buf base(u_in + ((size_t)lv * M + l) * W::N, u_end), add(c0 + (size_t)l * W::N, c0_end),
        o_buf(out + ((size_t)(r * 2 + p) * L + l) * W::N, out_end);
    whole_forward<LN>(xs, tw_a, tw_b, w, S);
#pragma unroll 1
    for (uint32_t it = threadIdx.x; it < G::IT4; it += W::T) {
      const uint32_t k2 = G::row4(it, true), o = G::off4(it, true), pos = G::pos_fwd(k2);
      uint64_t b[W::B::E2], a[W::B::E2];
#pragma unroll
      for (uint32_t u = 0; u < W::B::E2; ++u) {
        const Off ot = G::row(k2, o, u);
        b[u] = base.u64_once(ot.v, ot.s);
      }
      if (p == 0) {
#pragma unroll
        for (uint32_t u = 0; u < W::B::E2; ++u) {
          const Off on = G::natural(k2, o, u);
          a[u] = add.u64(on.v, on.s);
        }
      }
      double y[W::B::E2];
      whole_last<LN>(xs, pos, o, tw_b, y, S);
#pragma unroll
      for (uint32_t u = 0; u < W::B::E2; ++u) {
        double z = canonical(mul_tw(minuend<(W::B::kOut + 1 >= 4)>(b[u], y[u], q, qinv), S.inv, q), q, qinv);
        if (p == 0) {
          z += to_f64(a[u]);
          z = z >= q ? z - q : z;
        }
        xs[G::last_b(pos, o, u)] = z;
      }
    }
    __syncthreads();
#pragma unroll 4
    for (uint32_t d = threadIdx.x; d < W::N; d += W::T) {
      const uint32_t k = G::slot(gal, d);
      o_buf.put(to_u64(xs[G::word(G::pos_fwd(k % W::N2), k)]), G::dest(d), 0);
    }
    if (l + 1 < un.last) __syncthreads();
  }
}
#undef FIONA_WHOLE_KERNEL

// Groups that the n moduli of each of V vectors are split into: a workgroup
// takes one inverse and ceil(n / groups) forward transforms in turn, and the
// CUs run as many workgroups at once as eight waves each allow (at least one).
template <uint32_t LN>
uint32_t whole_groups(uint32_t V, uint32_t n) {
  constexpr uint32_t kCus = 256, waves = (Whole<LN>::T + 63) / 64, at_once = kCus * (waves < 8 ? 8 / waves : 1);
  uint32_t best = 1;
  uint64_t best_cost = ~0ull;
  for (uint32_t g = 1; g <= n; ++g) {
    const uint64_t chain = 1 + (n + g - 1) / g, turns = ((uint64_t)V * g + at_once - 1) / at_once;
    if (chain * turns < best_cost) {
      best_cost = chain * turns;
      best = g;
    }
  }
  return best;
}

}  // namespace fiona
