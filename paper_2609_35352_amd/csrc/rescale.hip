// Host side of the rescale epilogue (include/fiona.h): twiddle tables, the
// workspace and the launches of the NTT passes in ntt_kernel.hpp.
//
// Rescaling (paper Sec. 2, "Levels and Bootstrapping"; applied once per output
// after its routes are summed, Sec. 4.2 "Combining the Signed and Raw Routes")
// divides each coefficient's integer by the last modulus q_t = q_{L-1} with
// rounding.  In RNS form, for every other limb l:
//     out_l = (in_l - NTT_l([INTT_t(in_t)]_centred mod q_l)) * q_t^-1  mod q_l,
// where the centred remainder r in (-q_t/2, q_t/2] makes (C - r) / q_t the
// rounded quotient.  Only the last limb leaves the NTT domain.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "fiona.h"
#include "fiona_ctx.hpp"
#include "ntt_host.hpp"
#include "ntt_whole.hpp"

using namespace fiona_host;

// Intermediates of one launch pair, at most (chunk_size): the memory-side
// cache's 256 MiB.  Limits of 128 / 192 / 256 / 320 / 416 MiB and none, us:
// N = 2^16, L = 8, 128 ciphertexts 889 / 839 / 808 / 824 / 829 / 886; L = 16,
// 128: 1746 / 1659 / 1621 / 1640 / 1678 / 1811; L = 12, 96: 1024 / 933 / 923 /
// 916 / 942 / 1014; L = 32, 24: 714 / 644 / 627 / 615 / 632 / 660; N = 2^15,
// L = 16, 128: 890 / 850 / 812 / 819 / 835 / 923; N = 2^15, L = 8, 64 (one chunk
// from 256 on): 221 / 220 / 205 / 205 / 205 / 206.
constexpr size_t kTmpBytes = (size_t)256 << 20;

struct fiona_rescaler {
  const fiona_ctx *ctx = nullptr;
  uint32_t N = 0, L = 0, log_n1 = 0, log_n2 = 0, max_ct = 0;
  int device = -1;
  void *dev = nullptr;
  const NttSet *sets = nullptr;  // limbs 0 .. L-2 forward (inv = q_t^-1 mod q_l), then limb L-1 inverse
  double *W = nullptr;           // the centred remainders [INTT_t(in_t)] of a chunk, one vector per polynomial
  double *T = nullptr;           // the transposed intermediates of a chunk
  const void *W_end = nullptr, *T_end = nullptr;
};

namespace {

// Whether V vectors go as one launch of whole transforms (ntt_whole.hpp): up
// to N = 2^13 always; at 2^14, where a workgroup fills a CU, from 160 forward
// transforms on.  In passes / whole, us: L = 6, 4 ciphertexts (40 transforms)
// 21.0 / 28.9, 12 (120) 28.6 / 31.1, 16 (160) 32.9 / 32.1, 128 162 / 119; L = 16,
// 5 (150) 30.3 / 32.5, 6 (180) 34.5 / 33.7, 12 (360) 54.5 / 51.9, but 9 (270, one
// group too many for a turn of 256 workgroups) 45.3 / 48.6; L = 2, 60 (120)
// 36.7 / 31.6, 80 (160) 46.7 / 32.5.
constexpr uint32_t kWholeAlways = 13, kWholeMax = 14, kWholeTransforms = 160;
static_assert(kWholeAlways + 1 >= kPassMinLogN, "no passes are built for smaller rings");
bool use_whole(const fiona_rescaler *R, uint32_t V) {
  const uint32_t log_n = R->log_n1 + R->log_n2;
  return log_n <= kWholeAlways || (log_n <= kWholeMax && (uint64_t)V * (R->L - 1) >= kWholeTransforms);
}

// Bytes of a ciphertext's intermediates, and the ciphertexts of which a launch pair holds them.
size_t tmp_ct_bytes(const fiona_rescaler *R) {
  return (size_t)2 * (R->L - 1) * fiona::tmp_words(1u << R->log_n1, 1u << R->log_n2) * sizeof(double);
}
uint32_t chunk_max(const fiona_rescaler *R) {
  const size_t fit = kTmpBytes / tmp_ct_bytes(R);
  return fit < 1 ? 1 : fit < R->max_ct ? (uint32_t)fit : R->max_ct;
}

// Checks the parameters and sizes a rescaler: its tables (img) and the
// bytes of its device buffer (the table image, then W and T).
int rescaler_layout(const fiona_ctx *ctx, const uint64_t *psi, uint32_t max_ct, fiona_rescaler *R,
                    TableImage &img, size_t &total) {
  if (max_ct == 0) return FIONA_ERR_ARG;
  if (2ull * max_ct > 65535) return FIONA_ERR_UNSUPPORTED;   // (a transform takes two vectors a ciphertext)
  const uint32_t N = ctx->N, L = ctx->L;
  uint32_t logN = 0;
  while ((1u << logN) < N) ++logN;
  if ((1u << logN) != N || logN < 8 || logN > 17 || L < 2) return FIONA_ERR_UNSUPPORTED;
  std::vector<uint64_t> roots(L);
  for (uint32_t l = 0; l < L; ++l) {
    const uint64_t q = ctx->q[l];
    if ((q - 1) % (2ull * N) != 0) return FIONA_ERR_UNSUPPORTED;
    roots[l] = psi ? psi[l] % q : default_psi(N, q);
    if (roots[l] == 0 || powmod_h(roots[l], N, q) != q - 1) return FIONA_ERR_UNSUPPORTED;
  }
  R->ctx = ctx;
  R->N = N;
  R->L = L;
  R->log_n1 = (logN + 1) / 2;
  R->log_n2 = logN / 2;
  R->max_ct = max_ct;
  // every table of every limb and the set records, then the workspace
  const uint64_t qt = ctx->q[L - 1];
  for (uint32_t l = 0; l + 1 < L; ++l) {
    const uint64_t q = ctx->q[l];
    img.add(make_tables(R->log_n1, R->log_n2, q, roots[l], false), q, make_tw(powmod_h(qt % q, q - 2, q), q));
  }
  img.add(make_tables(R->log_n1, R->log_n2, qt, roots[L - 1], true), qt);
  const uint32_t chunk = chunk_max(R);
  total = img.bytes() + (logN <= kWholeAlways ? 0 : chunk * ((size_t)2 * N * sizeof(double) + tmp_ct_bytes(R)));
  return FIONA_OK;
}

// Points the rescaler's parts into its device buffer at dev.
void rescaler_place(fiona_rescaler *R, const TableImage &img, void *dev) {
  const size_t vec_bytes = (size_t)2 * chunk_max(R) * R->N * sizeof(double);
  R->dev = dev;
  R->sets = img.sets_addr(dev);
  R->W = (double *)((char *)dev + img.bytes());
  R->T = (double *)((char *)dev + img.bytes() + vec_bytes);
  if (R->log_n1 + R->log_n2 <= kWholeAlways) {   // no workspace: every call is whole
    R->W = R->T = nullptr;
    return;
  }
  R->W_end = (const char *)R->W + vec_bytes;
  R->T_end = (const char *)R->T + chunk_max(R) * tmp_ct_bytes(R);
}

void launch_whole(const fiona_rescaler *R, const uint64_t *in_cts, uint32_t V, uint64_t *out_cts, hipStream_t stream) {
  const uint32_t L = R->L;
  const size_t in_words = (size_t)V * L * R->N, out_words = (size_t)V * (L - 1) * R->N;
  for_log_n<kWholeMax>(R->log_n1 + R->log_n2, [&](auto ln) {
    constexpr uint32_t LN = decltype(ln)::value;
    const uint32_t groups = fiona::whole_groups<LN>(V, L - 1);
    if (LaunchRecord *rec = launch_recorder()) {
      rec->whole.push_back(WholeLaunch{WholeLaunch::kRescale, LN, V, L - 1, groups, in_cts, nullptr, out_cts,
                                       in_cts + in_words, nullptr, out_cts + out_words, R->sets + (L - 1), R->sets, {}});
      return;
    }
    hipLaunchKernelGGL(fiona::whole_rescale_kernel<LN>, dim3(V * groups), dim3(fiona::Whole<LN>::T),
                       fiona::whole_smem<LN>(), stream, in_cts, out_cts, R->sets, L, groups,
                       (const void *)(in_cts + in_words), (const void *)(out_cts + out_words));
  });
}

// The launches of one rescale (arguments already checked).
void rescale_enqueue(const fiona_rescaler *R, const uint64_t *in_cts, uint32_t n_ct, uint64_t *out_cts,
                     hipStream_t stream) {
  const size_t N = R->N, L = R->L;
  const uint32_t V = 2 * n_ct;
  if (use_whole(R, V)) return launch_whole(R, in_cts, V, out_cts, stream);
  const void *in_end = in_cts + (size_t)n_ct * 2 * L * N, *out_end = out_cts + (size_t)n_ct * 2 * (L - 1) * N;

  const uint32_t chunk = chunk_size(n_ct, kTmpBytes / tmp_ct_bytes(R));
  for (uint32_t c = 0; c < n_ct; c += chunk) {
    const uint32_t n = 2 * (n_ct - c < chunk ? n_ct - c : chunk);
    const uint64_t *in = in_cts + (size_t)c * 2 * L * N;
    const uint32_t nl = (uint32_t)L - 1;
    const bool nt = stores_nontemporal(R->log_n1, R->log_n2, nl * n);
    // 1. the last limb back to its coefficients, kept as centred residues mod q_t
    NttPass P{};
    P.sets = R->sets + (L - 1);
    P.vps = n;
    P.log_n1 = R->log_n1;
    P.log_n2 = R->log_n2;
    P.in = in + (L - 1) * N;
    P.in_end = in_end;
    P.in_stride = L * N;
    P.tmp = R->T;
    P.tmp_end = R->T_end;
    P.out = R->W;
    P.out_end = R->W_end;
    P.out_stride = N;
    P.load = fiona::kLoadU64;
    P.store = fiona::kStoreF64;
    P.nt = nt;
    launch_transform(R->log_n1, R->log_n2, n, stream, P);

    // 2. every other limb: the centred remainder (a signed integer, so its
    //    residue mod q_l comes with the first product) into its NTT domain,
    //    subtracted, multiplied by q_t^-1; all limbs in one launch pair (one
    //    set per limb, the vectors of a set share its modulus), pass A in the
    //    order that fetches each input block once per XCD
    NttPass Q{};
    Q.sets = R->sets;
    Q.vps = n;
    Q.log_n1 = R->log_n1;
    Q.log_n2 = R->log_n2;
    Q.in = R->W;
    Q.in_end = R->W_end;
    Q.in_stride = N;
    Q.tmp = R->T;
    Q.tmp_end = R->T_end;
    Q.out = out_cts + (size_t)c * 2 * (L - 1) * N;
    Q.out_end = out_end;
    Q.out_stride = (L - 1) * N;
    Q.out_set_stride = N;
    Q.base = in;
    Q.base_end = in_end;
    Q.base_stride = L * N;
    Q.base_set_stride = N;
    Q.load = fiona::kLoadF64;
    Q.store = fiona::kStoreRescale;
    Q.nt = nt;
    const uint32_t col_blocks = (1u << R->log_n1) / fiona::kNttCols;
    Q.nsets_shared = nl > 1 && (col_blocks * n) % 8 == 0 ? nl : 0;
    launch_transform(R->log_n1, R->log_n2, nl * n, stream, Q);
  }
}

}  // namespace

namespace fiona_host {

// A rescaler laid out at fake device addresses, one rescale of n_ct
// ciphertexts recorded and every access of its launches checked.  The
// caller's output region is out_shrink bytes short of its size (a check of
// the checker).
int rescale_replay(const uint64_t *moduli, uint32_t N, uint32_t L, uint32_t max_ct, uint32_t n_ct,
                   uint64_t out_shrink, std::string &err) {
  fiona_ctx *ctx = nullptr;
  int rc = fiona_ctx_create(N, L, moduli, &ctx);
  if (rc != FIONA_OK) return rc;
  fiona_rescaler R;
  TableImage img;
  size_t total = 0;
  rc = rescaler_layout(ctx, nullptr, max_ct, &R, img, total);
  if (rc == FIONA_OK && (n_ct == 0 || n_ct > max_ct)) rc = FIONA_ERR_ARG;
  if (rc != FIONA_OK) {
    fiona_ctx_destroy(ctx);
    return rc;
  }
  // separate fake allocations, 2^44 bytes apart
  // (each starts with bit 31 of its low address half set: the replay
  // rebuilds every descriptor base from its halves as the kernels do)
  const uint64_t kGap = 1ull << 44, kLow = 0x80000000ull;
  char *dev = (char *)(uintptr_t)(1 * kGap + kLow);
  const uint64_t *in = (const uint64_t *)(uintptr_t)(2 * kGap + kLow);
  uint64_t *out = (uint64_t *)(uintptr_t)(3 * kGap + kLow);
  rescaler_place(&R, img, dev);
  std::vector<Region> regions = table_regions(img, dev);
  regions.push_back(Region{(uint64_t)R.W, (uint64_t)R.W_end, "rescaler W"});
  regions.push_back(Region{(uint64_t)R.T, (uint64_t)R.T_end, "rescaler T"});
  regions.push_back(Region{(uint64_t)in, (uint64_t)(in + (size_t)n_ct * 2 * L * N), "in_cts"});
  regions.push_back(Region{(uint64_t)out, (uint64_t)(out + (size_t)n_ct * 2 * (L - 1) * N) - out_shrink, "out_cts"});
  LaunchRecord rec;
  launch_recorder() = &rec;
  rescale_enqueue(&R, in, n_ct, out, nullptr);
  launch_recorder() = nullptr;
  err = check_launches(rec, regions, (uint64_t)R.sets, img.sets_at(dev));
  fiona_ctx_destroy(ctx);
  return err.empty() ? FIONA_OK : FIONA_ERR_BOUNDS;
}

}  // namespace fiona_host

extern "C" {

int fiona_rescaler_create(const fiona_ctx *ctx, const uint64_t *psi, uint32_t max_ct, fiona_rescaler **out) {
  if (!out) return FIONA_ERR_ARG;
  *out = nullptr;
  if (!ctx) return FIONA_ERR_ARG;
  fiona_rescaler *R = new (std::nothrow) fiona_rescaler;
  if (!R) return FIONA_ERR_NOMEM;
  try {
    TableImage img;
    size_t total = 0;
    const int rc = rescaler_layout(ctx, psi, max_ct, R, img, total);
    if (rc != FIONA_OK) {
      delete R;
      return rc;
    }
    if (hipGetDevice(&R->device) != hipSuccess) {
      delete R;
      return FIONA_ERR_HIP;
    }
    void *dev = nullptr;
    if (hipMalloc(&dev, total) != hipSuccess) {
      delete R;
      return FIONA_ERR_NOMEM;
    }
    rescaler_place(R, img, dev);
    if (!img.upload(R->dev) || !allow_smem() ||
        !allow_lds((const void *)fiona::whole_rescale_kernel<13>, fiona::whole_smem<13>()) ||
        !allow_lds((const void *)fiona::whole_rescale_kernel<14>, fiona::whole_smem<14>())) {
      fiona_rescaler_destroy(R);
      return FIONA_ERR_HIP;
    }
  } catch (...) {
    fiona_rescaler_destroy(R);
    return FIONA_ERR_NOMEM;
  }
  *out = R;
  return FIONA_OK;
}

void fiona_rescaler_destroy(fiona_rescaler *R) {
  if (!R) return;
  if (R->dev) (void)hipFree(R->dev);
  delete R;
}

int fiona_rescale(const fiona_rescaler *R, const uint64_t *in_cts, uint32_t n_ct, uint64_t *out_cts,
                  hipStream_t stream) {
  if (!R) return FIONA_ERR_ARG;
  if (n_ct == 0) return FIONA_OK;
  if (!in_cts || !out_cts || n_ct > R->max_ct) return FIONA_ERR_ARG;
  if (((uintptr_t)in_cts | (uintptr_t)out_cts) & 7u) return FIONA_ERR_ALIGN;
  const size_t N = R->N, L = R->L;
  const size_t in_bytes = (size_t)n_ct * 2 * L * N * 8, out_bytes = (size_t)n_ct * 2 * (L - 1) * N * 8;
  const uintptr_t a0 = (uintptr_t)in_cts, b0 = (uintptr_t)out_cts;
  if (a0 < b0 + out_bytes && b0 < a0 + in_bytes) return FIONA_ERR_ALIAS;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != R->device) return FIONA_ERR_ARG;
  rescale_enqueue(R, in_cts, n_ct, out_cts, stream);
  if (hipGetLastError() != hipSuccess) return FIONA_ERR_HIP;
  return FIONA_OK;
}

}  // extern "C"
