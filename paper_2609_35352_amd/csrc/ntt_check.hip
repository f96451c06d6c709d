// Host replay of the NTT passes' memory accesses.
//
// A rescaler or rotator is laid out at fake device addresses, one call is
// recorded instead of launched (ntt_host.hpp), and every global access of
// every workgroup and thread of every recorded pass and launch of whole
// transforms is recomputed on the host through the same offset helpers the
// kernels use (GeomA, GeomB, GeomRot in ntt_kernel.hpp, GeomWhole in
// ntt_whole.hpp).  Each access must lie inside the buffer that holds its
// descriptor's base, every offset must stay below 2^32 bytes, and every
// descriptor's end pointer must be that buffer's end.  Of the whole
// transforms the LDS words are recomputed too: each step must touch every word
// of the vector once, inside the LDS.  No device is needed.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "fiona.h"
#include "ntt_host.hpp"
#include "ntt_whole.hpp"

namespace fiona_host {

namespace {

using fiona::DftShape;
using fiona::GeomA;
using fiona::GeomB;
using fiona::GeomRot;
using fiona::Off;
using fiona::kNttCols;

struct Checker {
  const std::vector<Region> &regions;
  uint64_t sets_dev;
  const std::vector<NttSet> &sets_host;
  std::string err, end_err;   // end_err: a descriptor end that differs (reported after the accesses)
  size_t launch = 0;

  const Region *find(uint64_t a) const {
    for (const Region &r : regions)
      if (a >= r.lo && a < r.hi) return &r;
    return nullptr;
  }
  bool fail(const std::string &m) {
    if (err.empty()) err = "launch " + std::to_string(launch) + ": " + m;
    return false;
  }
  // bytes [base + lo, base + hi) must lie in the region that holds base;
  // end (if not null) must be that region's end
  bool span(const char *what, uint64_t base, uint64_t lo, uint64_t hi, const void *end) {
    if (hi <= lo) return true;
    if (fiona::join_halves((uint32_t)(base >> 32), (uint32_t)base) != base)
      return fail(std::string(what) + ": base not rebuilt from its halves");
    const Region *r = find(base);
    if (!r) return fail(std::string(what) + ": base outside every buffer");
    if (base + hi > r->hi)
      return fail(std::string(what) + ": bytes up to " + std::to_string(base + hi - r->lo) + " of " + r->name +
                  " (" + std::to_string(r->hi - r->lo) + " bytes)");
    if (end && (uint64_t)end != r->hi && end_err.empty())
      end_err = "launch " + std::to_string(launch) + ": " + what + ": descriptor end differs from the end of " +
                r->name;
    return true;
  }
  // the largest end (offset + bytes) of accesses with offsets o, and the 2^32 limit
  bool grow(uint64_t &hi, Off o, uint32_t bytes, const char *what) {
    const uint64_t off = (uint64_t)o.v + o.s;
    if (off + bytes > 0xFFFFFFFFull) return fail(std::string(what) + ": offset beyond 2^32 bytes");
    hi = std::max(hi, off + bytes);
    return true;
  }
  const NttSet *set(const NttSet *p, uint32_t s) {
    const uint64_t a = (uint64_t)(p + s);
    if (a < sets_dev || (a - sets_dev) % sizeof(NttSet) != 0 || (a - sets_dev) / sizeof(NttSet) >= sets_host.size()) {
      fail("set record " + std::to_string(s) + " outside the NttSet array");
      return nullptr;
    }
    return &sets_host[(a - sets_dev) / sizeof(NttSet)];
  }
  bool tables(const Tw *dft, uint32_t n) {
    return span("transform twiddles", (uint64_t)dft, 0, (uint64_t)n * sizeof(Tw), nullptr);
  }
};

template <uint32_t LOGM>
bool pass_a(Checker &C, const PassLaunch &L) {
  using D = DftShape<LOGM>;
  using G = GeomA<LOGM>;
  const NttPass &P = L.P;
  const uint32_t N1 = 1u << P.log_n1, N2 = D::M, gx = N1 / kNttCols;
  if (P.log_n1 != L.log_other || N1 < kNttCols) return C.fail("pass A: bad sides");
  const bool trans = P.load == fiona::kLoadU64T, blocked = P.load == fiona::kLoadF64;
  // per column block: the largest ends of the accesses relative to each descriptor's base
  std::vector<uint64_t> in_hi(gx, 0), tmp_hi(gx, 0), mid_hi(gx, 0);
  for (uint32_t cb = 0; cb < gx; ++cb) {
    for (uint32_t it = 0; it < D::IT1; ++it) {
      const uint32_t cl = G::col(it, trans), ip = G::grp(it, trans), n1 = cb * kNttCols + cl;
      for (uint32_t u = 0; u < 16; ++u) {
        if (!C.grow(in_hi[cb], blocked ? G::in_b(cb, cl, ip, u) : trans ? G::in_t(n1, ip, u, N1) : G::in(n1, ip, u, N1),
                    8, "pass A input"))
          return false;
      }
    }
    for (uint32_t it = 0; it < D::IT2; ++it) {
      const uint32_t cl = G::col2(it), o = G::off2(it), n1 = cb * kNttCols + cl;
      for (uint32_t u = 0; u < D::E2; ++u)
        if (!C.grow(tmp_hi[cb], G::tmp(o, n1, u, N1), 8, "pass A tmp") ||
            !C.grow(mid_hi[cb], G::mid(cb, cl, o, u), 8, "pass A mid"))
          return false;
    }
  }
  for (uint32_t by = 0; by < L.V; ++by)
    for (uint32_t bx = 0; bx < gx; ++bx) {
      const fiona::UnitA un = fiona::pass_a_unit(P.vps, P.nsets_shared, bx, by, gx);
      const NttSet *S = C.set(P.sets, un.set);
      if (!S) return false;
      const uint64_t v = (uint64_t)un.set * P.vps + un.lv;
      const uint64_t in_base = (uint64_t)P.in + (un.set * P.in_set_stride + un.lv * P.in_stride) * 8;
      const uint64_t tmp_base = (uint64_t)P.tmp + v * fiona::tmp_words(N1, N2) * 8;
      if (!C.span("pass A input", in_base, 0, in_hi[un.cb], P.in_end) ||
          !C.span("pass A tmp", tmp_base, 0, tmp_hi[un.cb], P.tmp_end) ||
          !C.span("pass A mid", (uint64_t)S->mid, 0, mid_hi[un.cb], nullptr) ||
          !C.span("pass A mid table", (uint64_t)S->mid, 0, (uint64_t)N1 * N2 * sizeof(double), nullptr) ||
          !C.tables(S->dft_a, blocked ? D::M : D::M / 2))
        return false;
    }
  return true;
}

template <uint32_t LOGM>
bool pass_b(Checker &C, const PassLaunch &L) {
  using D = DftShape<LOGM>;
  using G = GeomB<LOGM>;
  const NttPass &P = L.P;
  const uint32_t M = D::M, N2 = 1u << P.log_n2, gx = N2 / kNttCols;
  if (P.log_n2 != L.log_other || N2 < kNttCols) return C.fail("pass B: bad sides");
  const bool transposed = P.store == fiona::kStoreU64T, rescale = P.store == fiona::kStoreRescale;
  uint64_t tmp_hi = 0;
  for (uint32_t it = 0; it < D::IT1; ++it)
    for (uint32_t u = 0; u < 16; ++u)
      if (!C.grow(tmp_hi, G::tmp(G::row(it), G::grp(it), u), 8, "pass B tmp")) return false;
  std::vector<uint64_t> out_hi(gx, 0), base_hi(gx, 0);
  uint64_t post_hi = 0;
  for (uint32_t x = 0; x < gx; ++x) {
    const uint32_t r0 = x * kNttCols;
    for (uint32_t it = 0; it < D::IT2; ++it) {
      const uint32_t row = G::row2(it, transposed), o = G::off2(it, transposed), k2 = r0 + row;
      for (uint32_t u = 0; u < D::E2; ++u) {
        if (!C.grow(post_hi, G::post(o, u), 16, "pass B post")) return false;
        const Off oc = G::col(k2, o, u, N2);
        if (rescale && !C.grow(base_hi[x], oc, 8, "pass B base")) return false;
        if (!C.grow(out_hi[x], transposed ? G::row_t(k2, o, u) : rescale ? oc : G::block(k2, o, u, N2), 8,
                    "pass B output"))
          return false;
      }
    }
  }
  for (uint32_t by = 0; by < L.V; ++by) {
    const fiona::UnitB un = fiona::pass_b_unit(P.vps, L.V, by);
    const uint32_t set = un.set, lv = un.lv;
    const NttSet *S = C.set(P.sets, set);
    if (!S || !C.tables(S->dft_b, D::M / 2)) return false;
    if (inverse_b(P) != (S->post != nullptr)) return C.fail("pass B: post table and direction differ");
    if (S->post && (!C.span("pass B post", (uint64_t)S->post, 0, post_hi, nullptr) ||
                    !C.span("pass B post table", (uint64_t)S->post, 0, (uint64_t)M * sizeof(Tw), nullptr)))
      return false;
    for (uint32_t x = 0; x < gx; ++x) {
      const uint64_t tmp_base = (uint64_t)P.tmp + (((uint64_t)set * P.vps + lv) * fiona::tmp_words(M, N2) +
                                                   (uint64_t)x * kNttCols * fiona::tmp_pitch(M)) * 8;
      const uint64_t out_base = (uint64_t)P.out + (set * P.out_set_stride + lv * P.out_stride) * 8;
      if (!C.span("pass B tmp", tmp_base, 0, tmp_hi, P.tmp_end) ||
          !C.span("pass B output", out_base, 0, out_hi[x], P.out_end))
        return false;
      if (rescale &&
          !C.span("pass B base", (uint64_t)P.base + (set * P.base_set_stride + lv * P.base_stride) * 8, 0, base_hi[x],
                  P.base_end))
        return false;
    }
  }
  return true;
}

template <uint32_t LOGM>
bool pass_b_rot(Checker &C, const PassLaunch &L) {
  using D = DftShape<LOGM>;
  using G = GeomRot<LOGM>;
  const NttPass &P = L.P;
  const RotArgs &R = L.G;
  const uint32_t N2 = 1u << P.log_n2, N = D::M << P.log_n2, gx = N2 / kNttCols;
  if (P.log_n2 != L.log_other || N2 < kNttCols || R.n_rot == 0 || R.n_rot > fiona::kRotMax)
    return C.fail("rotation pass B: bad shape");
  // per (column block, rotation): the rows read depend on the Galois element
  std::vector<uint64_t> tmp_hi((size_t)gx * R.n_rot, 0), word_hi((size_t)gx * R.n_rot, 0), add_hi((size_t)gx * R.n_rot, 0),
      out_hi(gx, 0);
  for (uint32_t x = 0; x < gx; ++x) {
    const uint32_t o0 = x * kNttCols;
    for (uint32_t r = 0; r < R.n_rot; ++r) {
      const uint32_t g = R.g[r];
      uint64_t &th = tmp_hi[(size_t)x * R.n_rot + r], &wh = word_hi[(size_t)x * R.n_rot + r],
               &ah = add_hi[(size_t)x * R.n_rot + r];
      for (uint32_t it = 0; it < D::IT1; ++it) {
        const uint32_t k2 = G::src_row(g, o0 + G::row(it), N2);
        for (uint32_t u = 0; u < 16; ++u)
          if (!C.grow(th, G::tmp(k2, G::grp(it), u), 8, "rotation pass B tmp")) return false;
      }
      for (uint32_t it = 0; it < D::IT2; ++it) {
        const uint32_t k2c = G::src_row(g, o0 + G::row2(it), N2);
        for (uint32_t u = 0; u < D::E2; ++u)
          if (!C.grow(wh, G::word(k2c, G::off2(it), u), 8, "rotation pass B u'") ||
              !C.grow(ah, R.c0_natural ? G::natural(k2c, G::off2(it), u, N2) : G::word(k2c, G::off2(it), u), 8,
                      "rotation pass B c0"))
            return false;
      }
    }
    for (uint32_t t = 0; t < fiona::kNttThreads; ++t)
      for (uint32_t j = 0; j < G::PER; ++j)
        if (!C.grow(out_hi[x], G::out(o0, t, j, N2), 8, "rotation pass B output")) return false;
  }
  for (uint32_t by = 0; by < L.V; ++by) {
    const fiona::UnitB un = fiona::pass_b_unit(P.vps, L.V, by);
    const uint32_t set = un.set, lv = un.lv, p = (R.lv0 + lv) / R.n_rot, r = R.lv0 + lv - p * R.n_rot;
    if (p > 1) return C.fail("rotation pass B: more than two polynomials per rotation");
    const NttSet *S = C.set(P.sets, set);
    if (!S || !C.tables(S->dft_b, D::M / 2)) return false;
    for (uint32_t x = 0; x < gx; ++x) {
      const size_t xr = (size_t)x * R.n_rot + r;
      if (!C.span("rotation pass B tmp", (uint64_t)P.tmp + ((uint64_t)set * P.vps + lv) * fiona::tmp_words(D::M, N2) * 8, 0, tmp_hi[xr], P.tmp_end) ||
          !C.span("rotation pass B u'", (uint64_t)P.base + (set * P.base_set_stride + lv * P.base_stride) * 8, 0,
                  word_hi[xr], P.base_end) ||
          (p == 0 && !C.span("rotation pass B c0", (uint64_t)P.add + set * P.add_set_stride * 8, 0, add_hi[xr],
                             P.add_end)) ||
          !C.span("rotation pass B output", (uint64_t)P.out + (((uint64_t)r * 2 + p) * R.L + set) * N * 8, 0,
                  out_hi[x], P.out_end))
        return false;
    }
  }
  return true;
}

// A set of N words, each to be met once.
struct Once {
  std::vector<uint8_t> seen;
  uint32_t left;
  explicit Once(uint32_t words, uint32_t n) : seen(words, 0), left(n) {}
  bool take(uint64_t w) {
    if (w >= seen.size() || seen[w] || !left) return false;
    seen[w] = 1;
    --left;
    return true;
  }
};

template <uint32_t LN>
bool whole(Checker &C, const WholeLaunch &L) {
  using W = fiona::Whole<LN>;
  using A = typename W::A;
  using B = typename W::B;
  using G = fiona::GeomWhole<LN>;
  constexpr uint32_t N = W::N;
  const bool trans = L.kind == WholeLaunch::kDivide, rowwise = L.kind != WholeLaunch::kRescale;
  const std::string name = L.kind == WholeLaunch::kRescale  ? "whole rescale"
                           : L.kind == WholeLaunch::kDigits ? "whole digits"
                                                            : "whole division";
  // one workgroup: the LDS words of each step (distinct, all N of them, inside
  // the vector's part of the LDS) and the offsets of each buffer (every word once)
  auto step = [&](const char *what, uint32_t words, uint32_t its, uint32_t per, auto index) {
    Once once(words, N);
    for (uint32_t it = 0; it < its; ++it)
      for (uint32_t u = 0; u < per; ++u)
        if (!once.take(index(it, u))) return C.fail(name + ": " + what + ": word met twice or outside");
    return once.left == 0 || C.fail(name + ": " + what + ": words left out");
  };
  auto bytes = [](Off o) { return ((uint64_t)o.v + o.s) % 8 ? ~0ull : ((uint64_t)o.v + o.s) / 8; };
  for (const bool fwd : {false, true})
    if (!step("first groups", W::WORDS, W::T, A::E1, [&](uint32_t t, uint32_t u) {
          const uint32_t n1 = G::col1(t), ip = G::grp1(t);
          return fwd ? G::first_fwd(n1, ip, u) : G::first_inv(n1, A::rev2(ip), u);
        }) ||
        !step("pass A's last groups", W::WORDS, G::IT2, A::E2, [&](uint32_t it, uint32_t e) {
          return G::last_a(G::col2(it), G::off2(it), A::rev1(G::off2(it)), e, fwd);
        }))
      return false;
  if (!step("pass B's reads", W::WORDS, G::IT3, B::E1,
            [&](uint32_t it, uint32_t u) { return G::b_in(G::pos3(it), G::grp3(it), u); }) ||
      !step("pass B's writes", W::WORDS, G::IT3, B::E1,
            [&](uint32_t it, uint32_t u) { return G::b_out(G::pos3(it), G::grp3(it), u); }) ||
      !step("coefficients", W::WORDS, W::T, A::E1, [&](uint32_t t, uint32_t v) {
        const uint32_t n = G::coef(G::col1(t), G::grp1(t), v);
        return G::word(n % W::N2, n);
      }))
    return false;
  for (const bool rw : {false, rowwise})   // the inverse's last groups, then the forward one's
    if (!step("last groups", W::WORDS, G::IT4, B::E2, [&](uint32_t it, uint32_t u) {
          const uint32_t k2 = G::row4(it, rw);
          return G::last_b(rw == rowwise ? G::pos_fwd(k2) : k2, G::off4(it, rw), u);
        }))
      return false;
  if (!step("input", N, W::T, A::E1,
            [&](uint32_t t, uint32_t u) { return bytes(Off{G::in(G::col1(t), G::grp1(t), u, trans), 0}); }) ||
      !step("mid", N, G::IT2, A::E2,
            [&](uint32_t it, uint32_t u) { return bytes(G::mid(G::col2(it), G::off2(it), u)); }) ||
      !step("natural order", N, G::IT4, B::E2, [&](uint32_t it, uint32_t u) {
        return bytes(G::natural(G::row4(it, rowwise), G::off4(it, rowwise), u));
      }))
    return false;
  if (rowwise && !step("transposed", N, G::IT4, B::E2, [&](uint32_t it, uint32_t u) {
        return bytes(G::row(G::row4(it, true), G::off4(it, true), u));
      }))
    return false;
  uint64_t post_hi = 0;
  for (uint32_t it = 0; it < G::IT4; ++it)
    for (uint32_t u = 0; u < B::E2; ++u)
      if (!C.grow(post_hi, G::post(G::off4(it, false), u), 16, "whole transform post")) return false;
  if (trans)
    for (uint32_t r = 0; r < L.G.n_rot; ++r)
      if (!step("automorphism's reads", W::WORDS, N, 1, [&](uint32_t d, uint32_t) {
            const uint32_t k = G::slot(L.G.g[r], d);
            return G::word(G::pos_fwd(k % W::N2), k);
          }) ||
          !step("automorphism's writes", N, N, 1, [&](uint32_t d, uint32_t) { return bytes(Off{G::dest(d), 0}); }))
        return false;

  // every workgroup: its buffers and tables, each output vector once
  constexpr uint64_t vec = (uint64_t)N * 8;
  auto tables = [&](const NttSet *S, bool fwd) {
    return S && (fwd == (S->post == nullptr) || C.fail(name + ": post table and direction differ")) &&
           C.span("whole transform mid", (uint64_t)S->mid, 0, vec, nullptr) &&
           C.tables(S->dft_a, fwd ? W::N2 : W::N2 / 2) && C.tables(S->dft_b, W::N1 / 2) &&
           (fwd || C.span("whole transform post", (uint64_t)S->post, 0, post_hi, nullptr));
  };
  const uint32_t in_vec = L.kind == WholeLaunch::kDigits ? 1 : L.n + 1;   // vectors per input vector: all its limbs
  Once outs(L.V * L.n, L.V * L.n);
  for (uint32_t b = 0; b < L.V * L.groups; ++b) {
    const fiona::WholeUnit un = fiona::whole_unit(b, L.groups, L.n);
    if (un.v >= L.V || un.last > L.n) return C.fail(name + ": workgroup outside the call");
    const uint64_t in = (uint64_t)L.in + un.v * in_vec * vec;
    const NttSet *I = C.set(L.inv_sets, L.kind == WholeLaunch::kDigits ? un.v : 0);
    if (!tables(I, false)) return false;
    const uint64_t inv_at = in + (in_vec - 1) * vec;   // the limb that goes back to its coefficients
    const std::string at = name + ", vector " + std::to_string(un.v);
    if (!C.span((at + ": input").c_str(), inv_at, 0, vec, L.in_end)) return false;
    for (uint32_t l = un.first; l < un.last; ++l) {
      const std::string atl = at + ", modulus " + std::to_string(l);
      if (!tables(C.set(L.fwd_sets, l), true)) return false;
      uint64_t o = (uint64_t)un.v * L.n + l;   // the output vector
      if (L.kind == WholeLaunch::kDivide) {
        const uint32_t p = un.v / L.G.n_rot, r = un.v - p * L.G.n_rot;
        if (p > 1 || L.G.L != L.n) return C.fail(atl + ": bad shape");
        o = ((uint64_t)r * 2 + p) * L.n + l;
        if (p == 0 && !C.span((atl + ": c0").c_str(), (uint64_t)L.add + l * vec, 0, vec, L.add_end)) return false;
      }
      if (L.kind != WholeLaunch::kDigits && !C.span((atl + ": minuends").c_str(), in + l * vec, 0, vec, L.in_end))
        return false;
      if (!C.span((atl + ": output").c_str(), (uint64_t)L.out + o * vec, 0, vec, L.out_end)) return false;
      if (!outs.take(o)) return C.fail(atl + ": output written twice");
    }
  }
  return outs.left == 0 || C.fail(name + ": outputs left out");
}

}  // namespace

std::string check_launches(const LaunchRecord &rec, const std::vector<Region> &regions, uint64_t sets_dev,
                           const std::vector<NttSet> &sets_host) {
  Checker C{regions, sets_dev, sets_host, std::string()};
  for (const LdsUse &u : rec.lds)
    if (u.bytes > u.most)
      return std::string(u.what) + ": " + std::to_string(u.bytes) + " bytes of LDS, its limit is " +
             std::to_string(u.most);
  for (const SpanAccess &s : rec.spans)
    if (!C.span(s.what, s.base, s.lo, s.hi, nullptr)) return C.err;
  for (const WholeLaunch &L : rec.whole) {
    if (L.V == 0 || L.groups == 0 || L.groups > L.n) {
      C.fail("bad whole launch");
      return C.err;
    }
    bool ok = false;
    for_log_n<14>(L.log_n, [&](auto ln) { ok = whole<decltype(ln)::value>(C, L); });
    if (!ok) return C.err.empty() ? "whole launch outside 2^8 .. 2^14" : C.err;
    ++C.launch;
  }
  for (const PassLaunch &L : rec.passes) {
    if (L.V == 0 || L.V > 65535 || L.P.vps == 0) {
      C.fail("bad vector count");
      return C.err;
    }
    bool ok = false;
    if (L.kind == PassLaunch::kPassA)
      for_log_n<kSideMaxA, kSideMinA>(L.log_side, [&](auto ls) { ok = pass_a<decltype(ls)::value>(C, L); });
    else
      for_log_n<kSideMaxB, kSideMinB>(L.log_side, [&](auto ls) {
        constexpr uint32_t LOG = decltype(ls)::value;
        ok = L.kind == PassLaunch::kPassB ? pass_b<LOG>(C, L) : pass_b_rot<LOG>(C, L);
      });
    if (!ok && C.err.empty()) C.fail("DFT side of no kernel");
    if (!ok) return C.err;
    ++C.launch;
  }
  return C.end_err;
}

}  // namespace fiona_host

extern "C" int fiona_check_ntt_offsets(uint32_t op, uint32_t N, uint32_t L, const uint64_t *moduli,
                                       uint32_t capacity, uint32_t n_call, uint64_t out_shrink, char *msg,
                                       size_t msg_len) {
  if (!moduli || op > 1) return FIONA_ERR_ARG;
  std::string err;
  int rc;
  try {
    rc = op == 0 ? fiona_host::rescale_replay(moduli, N, L, capacity, n_call, out_shrink, err)
                 : fiona_host::rotate_replay(moduli, N, L, capacity, n_call, out_shrink, err);
  } catch (...) {
    return FIONA_ERR_NOMEM;
  }
  if (msg && msg_len) {
    std::strncpy(msg, err.c_str(), msg_len - 1);
    msg[msg_len - 1] = '\0';
  }
  return rc;
}
