// Deep-pipelined GEMM instantiations per operand layout and epilogue: the 128 x 128 tile on 8 wavefronts with five K tiles in LDS, the
// same with two (64 KiB: two workgroups on a compute unit, one's stores and first loads under the other's products), 128 x 256 with three, and
// 64 x 64 on 4 wavefronts with three.
#include "ntp_gemm_launch.h"

#include "ntp_gemm_deep.h"

namespace ntp_gemm {

namespace {

template <bool AKC, bool BKC, int EPI, int BM_, int BN_, int WGM, int WGN, int STAGES>
int launch_tile(GemmArgs g, hipStream_t s) {
  g.tiles_m = (g.M + BM_ - 1) / BM_;
  g.tiles_n = (g.n_store + BN_ - 1) / BN_;
  const int64_t per_split = (int64_t(g.tiles_m) * g.tiles_n + 7) / 8 * 8;
  if (g.k_splits < 1 || g.k_chunk < 64 || g.k_chunk % 64 || int64_t(g.k_splits - 1) * g.k_chunk >= g.K || per_split * g.k_splits > 0x7fffffff)
    return NTP_ERR_INVALID_ARG;
  hipLaunchKernelGGL((gemm_deep_kernel<AKC, BKC, EPI, BM_, BN_, WGM, WGN, STAGES>), dim3(uint32_t(per_split * g.k_splits)), dim3(64 * WGM * WGN), 0, s, g);
  return hipGetLastError() == hipSuccess ? NTP_OK : NTP_ERR_LAUNCH;
}

template <bool AKC, bool BKC, int EPI>
int launch_one(const GemmArgs& g, int form, hipStream_t s) {
  switch (form) {
    case kDeep5: return launch_tile<AKC, BKC, EPI, 128, 128, 2, 4, 5>(g, s);
    case kDeep2: return launch_tile<AKC, BKC, EPI, 128, 128, 2, 4, 2>(g, s);
    case kDeepWide: return launch_tile<AKC, BKC, EPI, 128, 256, 2, 4, 3>(g, s);
    case kDeepSmall: return launch_tile<AKC, BKC, EPI, 64, 64, 2, 2, 3>(g, s);
    default: return NTP_ERR_INVALID_ARG;
  }
}

}  // namespace

int launch_deep(const GemmArgs& g, bool a_kc, bool b_kc, int epilogue, int form, hipStream_t s) {
  if (g.k_splits > 1) epilogue = ntp::EPI_F32;  // partial sums
  if (a_kc && b_kc) {
    switch (epilogue) {
      case ntp::EPI_BF16: return launch_one<true, true, ntp::EPI_BF16>(g, form, s);
      case ntp::EPI_GELU: return launch_one<true, true, ntp::EPI_GELU>(g, form, s);
      case ntp::EPI_DGELU: return launch_one<true, true, ntp::EPI_DGELU>(g, form, s);
      case ntp::EPI_F32: return launch_one<true, true, ntp::EPI_F32>(g, form, s);
    }
  } else if (a_kc) {
    switch (epilogue) {
      case ntp::EPI_BF16: return launch_one<true, false, ntp::EPI_BF16>(g, form, s);
      case ntp::EPI_F32: return launch_one<true, false, ntp::EPI_F32>(g, form, s);
    }
  } else if (!b_kc) {
    switch (epilogue) {
      case ntp::EPI_F32: return launch_one<false, false, ntp::EPI_F32>(g, form, s);
      case ntp::EPI_F32_ACCUM: return launch_one<false, false, ntp::EPI_F32_ACCUM>(g, form, s);
    }
  }
  return NTP_ERR_UNSUPPORTED;
}

int launch_deep_group(const GemmArgs* g, const int* layout, const int* epilogue, int n, int form, hipStream_t s) {
  const int b = form == kDeepSmall ? 64 : 128;
  if (n < 1 || n > kMaxGroup) return NTP_ERR_INVALID_ARG;
  GroupArgs a{};
  int64_t blocks = 0;
  for (int i = 0; i < n; ++i) {
    a.g[i] = g[i];
    a.g[i].tiles_m = (g[i].M + b - 1) / b;
    a.g[i].tiles_n = (g[i].n_store + b - 1) / b;
    if (layout[i] == 2 ? epilogue[i] != ntp::EPI_F32 && epilogue[i] != ntp::EPI_F32_ACCUM : epilogue[i] != ntp::EPI_BF16) return NTP_ERR_UNSUPPORTED;
    a.kind[i] = layout[i] == 0 ? kGroupNt : layout[i] == 1 ? kGroupNn : epilogue[i] == ntp::EPI_F32 ? kGroupTn : kGroupTnAccum;
    a.first[i] = int32_t(blocks);
    blocks += (int64_t(a.g[i].tiles_m) * a.g[i].tiles_n + 7) / 8 * 8;
    if (blocks > 0x7fffffff) return NTP_ERR_UNSUPPORTED;
  }
  a.n = n;
  if (form == kDeepSmall) hipLaunchKernelGGL((gemm_deep_group_kernel<64, 2, 3>), dim3(uint32_t(blocks)), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((gemm_deep_group_kernel<128, 4, 5>), dim3(uint32_t(blocks)), dim3(512), 0, s, a);
  return hipGetLastError() == hipSuccess ? NTP_OK : NTP_ERR_LAUNCH;
}

}  // namespace ntp_gemm
