// Host side of the NTT passes (ntt_kernel.hpp): twiddle tables, the table
// image in device memory, and the launch of one pass.  Shared by the rescale
// epilogue (rescale.hip) and the rotation producer (rotate.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "ntt_kernel.hpp"

namespace fiona_host {

using fiona::NttPass;
using fiona::NttSet;
using fiona::RotArgs;
using fiona::Tw;

// A launch as the host replay sees it (ntt_check.hip).  With a recorder
// installed, the launch helpers below record their launches instead of
// issuing them; the other kernels of a call record the byte ranges they
// touch.
struct PassLaunch {
  enum Kind : uint32_t { kPassA, kPassB, kPassBRot } kind;
  uint32_t log_side, log_other, V;   // DFT side, the other side, vectors (gridDim.y)
  NttPass P;
  RotArgs G;                         // kPassBRot only
};
// A launch of whole transforms (ntt_whole.hpp): V vectors, each with n moduli in groups.
struct WholeLaunch {
  enum Kind : uint32_t { kRescale, kDigits, kDivide } kind;
  uint32_t log_n, V, n, groups;
  const uint64_t *in, *add;   // kDivide: u' and c0
  uint64_t *out;
  const void *in_end, *add_end, *out_end;
  const NttSet *inv_sets, *fwd_sets;
  RotArgs G;                  // kDivide only
};
struct SpanAccess {   // another kernel: bytes [lo, hi) of the buffer at base
  const char *what;
  uint64_t base, lo, hi;
};
struct LdsUse {   // the LDS a launch asks for, and the most its kernel may
  const char *what;
  uint64_t bytes, most;
};
struct LaunchRecord {
  std::vector<PassLaunch> passes;
  std::vector<WholeLaunch> whole;
  std::vector<SpanAccess> spans;
  std::vector<LdsUse> lds;
};
inline LaunchRecord *&launch_recorder() {
  static thread_local LaunchRecord *rec = nullptr;
  return rec;
}
inline bool record_span(const char *what, const void *base, uint64_t lo, uint64_t hi) {
  LaunchRecord *rec = launch_recorder();
  if (!rec) return false;
  rec->spans.push_back(SpanAccess{what, (uint64_t)base, lo, hi});
  return true;
}

// A buffer of the replayed layout: bytes [lo, hi) of a fake address space.
struct Region {
  uint64_t lo, hi;
  std::string name;
};
// Checks every access of the recorded launches: each must fall inside the
// region that holds its descriptor's base, and each descriptor's end pointer
// must be that region's end.  sets_dev / sets_host: the device address of
// the table image's NttSet array and its host copy.  Returns "" or the
// first violation.
std::string check_launches(const LaunchRecord &rec, const std::vector<Region> &regions, uint64_t sets_dev,
                           const std::vector<NttSet> &sets_host);
// The replays of a rescale and of a rotation call (rescale.hip, rotate.hip).
int rescale_replay(const uint64_t *moduli, uint32_t N, uint32_t L, uint32_t max_ct, uint32_t n_ct,
                   uint64_t out_shrink, std::string &err);
int rotate_replay(const uint64_t *moduli, uint32_t N, uint32_t L, uint32_t max_rot, uint32_t n_rot,
                  uint64_t out_shrink, std::string &err);

inline uint64_t mulmod_h(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((unsigned __int128)a * b % q); }

inline uint64_t powmod_h(uint64_t b, uint64_t e, uint64_t q) {
  uint64_t r = 1 % q;
  b %= q;
  while (e) {
    if (e & 1) r = mulmod_h(r, b, q);
    b = mulmod_h(b, b, q);
    e >>= 1;
  }
  return r;
}

// The centred twiddle of w in [0, q).
inline Tw make_tw(uint64_t w, uint64_t q) {
  const double c = w > q / 2 ? -(double)(q - w) : (double)w;
  return Tw{c, c / (double)q};
}

// The default root: psi = x^((q-1)/2N) for the smallest x >= 2 with psi^N = -1.
inline uint64_t default_psi(uint32_t N, uint64_t q) {
  for (uint64_t x = 2; x < 1000000; ++x) {
    const uint64_t psi = powmod_h(x, (q - 1) / (2ull * N), q);
    if (powmod_h(psi, N, q) == q - 1) return psi;
  }
  return 0;
}

inline double centred(uint64_t w, uint64_t q) { return make_tw(w, q).w; }

// Tables of one direction of one modulus, for n = n1 + N1 n2 on the input
// side and k = k2 + N2 k1 on the output side (see ntt_kernel.hpp).  Forward:
// dft_a[2^s + b] = phi^bitrev(2^s + b) with phi = psi^N1 (N2 entries, the
// first unused), and the factor psi^n1, constant along pass A's transform,
// joins mid = omega^(n1 k2) psi^n1 (in pass A's column blocks, see NttSet).
// Inverse (omega -> omega^-1): dft_a the DFT twiddles of root omega^N1 (N2 /
// 2); the factor N^-1 psi^-k = N^-1 psi^-k2 psi^(-N2 k1): the part in k2,
// constant along pass B's DFT, joins mid = omega^(-n1 k2) N^-1 psi^-k2, and
// post = psi^(-N2 k1) (N1 entries).  dft_b: the DFT twiddles of root omega^N2.
struct TableSet {
  std::vector<Tw> dft_a, dft_b, post;
  std::vector<double> mid;
};

inline TableSet make_tables(uint32_t log_n1, uint32_t log_n2, uint64_t q, uint64_t psi, bool inverse) {
  const uint32_t N1 = 1u << log_n1, N2 = 1u << log_n2, N = N1 * N2;
  const uint64_t psi_inv = powmod_h(psi, q - 2, q);
  const uint64_t omega = inverse ? mulmod_h(psi_inv, psi_inv, q) : mulmod_h(psi, psi, q);
  TableSet t;
  auto powers = [&](std::vector<Tw> &v, size_t n, uint64_t step) {
    v.resize(n);
    uint64_t p = 1;
    for (size_t i = 0; i < n; ++i, p = mulmod_h(p, step, q)) v[i] = make_tw(p, q);
  };
  if (inverse) {
    powers(t.post, N1, powmod_h(psi_inv, N2, q));
    powers(t.dft_a, N2 / 2, powmod_h(omega, N1, q));
  } else {
    std::vector<Tw> phi;
    powers(phi, N2, powmod_h(psi, N1, q));
    t.dft_a.resize(N2);
    for (uint32_t i = 0; i < N2; ++i) {
      uint32_t r = 0;
      for (uint32_t b = 0; b < log_n2; ++b) r |= ((i >> b) & 1u) << (log_n2 - 1 - b);
      t.dft_a[i] = phi[r];
    }
  }
  powers(t.dft_b, N1 / 2, powmod_h(omega, N2, q));
  t.mid.resize(N);
  const uint32_t cols = fiona::kNttCols;
  const uint64_t n_inv = powmod_h(N, q - 2, q);
  for (uint32_t n1 = 0; n1 < N1; ++n1) {
    const uint64_t step = powmod_h(omega, n1, q), mul = inverse ? mulmod_h(step, psi_inv, q) : step;
    uint64_t p = inverse ? n_inv : powmod_h(psi, n1, q);   // the k2 = 0 entry
    for (uint32_t k2 = 0; k2 < N2; ++k2, p = mulmod_h(p, mul, q))
      t.mid[((size_t)(n1 / cols) * N2 + k2) * cols + n1 % cols] = centred(p, q);
  }
  return t;
}

// Host image of table sets: all tables back to back (in doubles), then the
// NttSet records, which point into the device copy of the same image.
struct TableImage {
  std::vector<double> words;
  struct Entry {
    size_t mid, dft_a, dft_b, post;
    uint64_t q;
    Tw inv;
  };
  static constexpr size_t kNone = (size_t)-1;
  std::vector<Entry> entries;

  // Appends the tables of one modulus; returns its set index.
  uint32_t add(const TableSet &t, uint64_t q, Tw inv = Tw{0.0, 0.0}) {
    auto put = [&](const auto &v) {
      const size_t o = words.size(), n = v.size() * sizeof(v[0]) / sizeof(double);
      if (!n) return kNone;
      words.resize(o + n);   // (every table is an even number of doubles: the twiddle pairs stay aligned)
      std::memcpy(&words[o], v.data(), n * sizeof(double));
      return o;
    };
    Entry e{put(t.mid), put(t.dft_a), put(t.dft_b), put(t.post), q, inv};
    entries.push_back(e);
    return (uint32_t)entries.size() - 1;
  }

  size_t table_bytes() const { return (words.size() * sizeof(double) + 255) / 256 * 256; }
  size_t bytes() const { return table_bytes() + (entries.size() * sizeof(NttSet) + 255) / 256 * 256; }

  // The NttSet records of an image placed at device address dev.
  std::vector<NttSet> sets_at(const void *dev) const {
    const double *tb = (const double *)dev;
    auto at = [&](size_t o) { return o == kNone ? nullptr : tb + o; };
    std::vector<NttSet> sets;
    for (const Entry &e : entries)
      sets.push_back(NttSet{at(e.mid), (const Tw *)at(e.dft_a), (const Tw *)at(e.dft_b), (const Tw *)at(e.post), e.inv,
                            (double)e.q, 1.0 / (double)e.q});
    return sets;
  }
  NttSet *sets_addr(void *dev) const { return (NttSet *)((char *)dev + table_bytes()); }

  // Copies the image to dev (bytes() long); returns the device NttSet array.
  NttSet *upload(void *dev) const {
    const std::vector<NttSet> sets = sets_at(dev);
    NttSet *dsets = sets_addr(dev);
    if (hipMemcpy(dev, words.data(), words.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess)
      return nullptr;
    if (hipMemcpy(dsets, sets.data(), sets.size() * sizeof(NttSet), hipMemcpyHostToDevice) != hipSuccess)
      return nullptr;
    return dsets;
  }
};

// The regions of an image placed at dev: each table of each set on its own,
// then the NttSet array.
inline std::vector<Region> table_regions(const TableImage &img, const void *dev) {
  std::vector<Region> r;
  const uint64_t base = (uint64_t)dev;
  const size_t n = img.words.size();
  for (size_t s = 0; s < img.entries.size(); ++s) {
    const TableImage::Entry &e = img.entries[s];
    const size_t offs[4] = {e.mid, e.dft_a, e.dft_b, e.post};
    const char *names[4] = {"mid", "dft_a", "dft_b", "post"};
    for (int t = 0; t < 4; ++t) {
      if (offs[t] == TableImage::kNone) continue;
      size_t end = n;   // the next table's start, else the end of the tables
      for (const TableImage::Entry &f : img.entries) {
        const size_t o2[4] = {f.mid, f.dft_a, f.dft_b, f.post};
        for (size_t o : o2)
          if (o != TableImage::kNone && o > offs[t] && o < end) end = o;
      }
      r.push_back(Region{base + offs[t] * sizeof(double), base + end * sizeof(double),
                         "set " + std::to_string(s) + " " + names[t]});
    }
  }
  r.push_back(Region{base + img.table_bytes(), base + img.table_bytes() + img.entries.size() * sizeof(NttSet),
                     "NttSet records"});
  return r;
}

// f(integral_constant<uint32_t, log_n>) for 8 <= log_n <= MAX.
template <uint32_t MAX, uint32_t LN = 8, typename F>
void for_log_n(uint32_t log_n, F &&f) {
  if (log_n == LN) f(std::integral_constant<uint32_t, LN>());
  else if constexpr (LN < MAX) for_log_n<MAX, LN + 1>(log_n, f);
}

// Lets a kernel use bytes of dynamic LDS.
inline bool allow_lds(const void *kernel, size_t bytes) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
}

// Whether a pass B ends an inverse transform.
inline bool inverse_b(const NttPass &P) { return P.store == fiona::kStoreF64 || P.store == fiona::kStoreF64C; }

// The passes run from N = 2^13 on (smaller rings go as whole transforms): pass A
// over sides N2 = 2^6 .. 2^8, pass B over N1 = 2^7 .. 2^9.
constexpr uint32_t kPassMinLogN = 13, kSideMinA = 6, kSideMaxA = 8, kSideMinB = 7, kSideMaxB = 9;

template <uint32_t LOG>
auto *pass_a_kernel(const NttPass &P) {
  if (P.load == fiona::kLoadF64) return P.nt ? fiona::ntt_pass_a<LOG, true, true> : fiona::ntt_pass_a<LOG, true, false>;
  return P.nt ? fiona::ntt_pass_a<LOG, false, true> : fiona::ntt_pass_a<LOG, false, false>;
}
template <uint32_t LOG>
auto *pass_b_kernel(const NttPass &P) {
  if (inverse_b(P)) return P.nt ? fiona::ntt_pass_b<LOG, true, true> : fiona::ntt_pass_b<LOG, true, false>;
  return fiona::ntt_pass_b<LOG, false, false>;   // stores no doubles
}

// LDS of a pass of side M: the columns and at most M twiddles.
constexpr size_t pass_smem(uint32_t M) {
  return fiona::kNttCols * fiona::padded_len(M) * sizeof(double) + M * sizeof(Tw);
}

// A call whose intermediates pass a limit (the rescale's and the division's
// own) goes in chunks, each with its launches, so that pass B finds pass A's
// words in the memory-side cache and the next chunk overwrites them there.
// The chunk size of n vectors (or pairs) of which `fit` are within the limit:
// as few chunks as that allows, of equal size.
inline uint32_t chunk_size(uint32_t n, size_t fit) {
  const uint32_t most = fit < 1 ? 1 : fit > n ? n : (uint32_t)fit, chunks = (n + most - 1) / most;
  return (n + chunks - 1) / chunks;
}

// Whether the two transforms of a step (the inverse one, then the forward one
// over V vectors, the larger) store their doubles nontemporally.  With the
// default policy the 256 MiB memory-side cache keeps them for the pass that
// reads them: a loop of writes and reads over 128 MiB moves 7.1 TB/s, with
// nontemporal stores 5.6, over 1 GiB 5.4 and 5.2.  But what a launch leaves in
// the L2s (8 of 4 MiB) is written back at its end, with nothing else in flight,
// which launches of one or two turns of workgroups pay for; with few words
// there is little to write back.  Default / nontemporal, us, by the forward
// intermediates' MiB, rescales: 2.1 (N = 2^16, L = 3, 1 ciphertext) 22.1 / 22.6,
// 4.2 (2^16, L = 2, 4) 24.3 / 23.4, 13 (2^15, L = 3, 12) 33.9 / 30.1, 21 (2^16,
// L = 6, 4) 38.9 / 35.4, 32 (2^15, L = 6, 12; 2^16, L = 16, 2) 46.3 / 46.3 and
// 43.9 / 41.3, 34 (2^15, L = 3, 32; 2^17, L = 2, 16) 53.4 / 52.9 and 68.6 /
// 67.8, 43 (2^15, L = 6, 16) 53.3 / 57.1, 64 (2^16, L = 16, 4) 64.0 / 66.9, 272
// (2^15, L = 6, 64) 149 / 175; rotations: 17 (2^15, L = 2, 16) 79.5 / 76.3, 27
// (2^14, L = 4, 24) 94.8 / 92.8 (but 28 at L = 1, 100 of 2^14, 120 / 125), 42
// (2^15, L = 2, 40) 143 / 145.  One policy for both transforms: a small inverse
// launch beside a large forward one loses with nontemporal stores (2^16, L = 8,
// 128 ciphertexts 822 -> 892).
inline bool stores_nontemporal(uint32_t log_n1, uint32_t log_n2, uint32_t V) {
  const size_t bytes = V * fiona::tmp_words(1u << log_n1, 1u << log_n2) * sizeof(double);
  return bytes >= (size_t)4 << 20 && bytes <= (size_t)32 << 20;
}

// One pass over gridDim.y = V vectors (V <= 65535).
inline void launch_pass(bool a, uint32_t log_side, uint32_t log_other, uint32_t V, hipStream_t stream,
                        const NttPass &P) {
  if (LaunchRecord *rec = launch_recorder()) {
    rec->passes.push_back(PassLaunch{a ? PassLaunch::kPassA : PassLaunch::kPassB, log_side, log_other, V, P, {}});
    return;
  }
  const dim3 grid((1u << log_other) / fiona::kNttCols, V);
  const size_t smem = pass_smem(1u << log_side);
  const dim3 block(fiona::kNttThreads);
  if (a)
    for_log_n<kSideMaxA, kSideMinA>(
        log_side, [&](auto ls) { hipLaunchKernelGGL(pass_a_kernel<decltype(ls)::value>(P), grid, block, smem, stream, P); });
  else
    for_log_n<kSideMaxB, kSideMinB>(
        log_side, [&](auto ls) { hipLaunchKernelGGL(pass_b_kernel<decltype(ls)::value>(P), grid, block, smem, stream, P); });
}

// Both passes of one transform.
inline void launch_transform(uint32_t log_n1, uint32_t log_n2, uint32_t V, hipStream_t stream, const NttPass &P) {
  launch_pass(true, log_n2, log_n1, V, stream, P);
  launch_pass(false, log_n1, log_n2, V, stream, P);
}

// Lets pass B over its largest side use its LDS (the other passes' fits the
// default of 64 KiB).
static_assert(pass_smem(1u << kSideMaxA) <= 64 * 1024 && pass_smem(1u << (kSideMaxB - 1)) <= 64 * 1024, "allow_smem");
inline bool allow_smem() {
  constexpr size_t smem = pass_smem(1u << kSideMaxB);
  return allow_lds((const void *)fiona::ntt_pass_b<kSideMaxB, true, true>, smem) &&
         allow_lds((const void *)fiona::ntt_pass_b<kSideMaxB, true, false>, smem) &&
         allow_lds((const void *)fiona::ntt_pass_b<kSideMaxB, false, false>, smem);
}

}  // namespace fiona_host
