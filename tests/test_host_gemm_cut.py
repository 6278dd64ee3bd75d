"""When a contraction axis is cut (no GPU): the number of chunks, which fixes the order of a product's fp32 sums, and what hangs on the same choice, the
workspace that the library asks for and the shapes that the call with static scratch refuses."""
import os
import shutil
import subprocess

import pytest

import paper_2504_06095_amd as N
from paper_2504_06095_amd import binding as Bd
from paper_2504_06095_amd import build

FAKE_WS = 0x10000000  # an aligned address: registering touches no memory


@pytest.fixture
def handle():
    h = Bd.ntp_create()
    assert Bd.lib().ntp_set_workspace(h.ptr, FAKE_WS, 1 << 32) == 0
    yield h
    assert Bd.lib().ntp_set_workspace(h.ptr, None, 0) == 0
    Bd.ntp_destroy(h)


# the projections of an attention shard of three heads, MLP halves of narrow shards, and products a little above one 128 x 128 tile per compute unit,
# which run whole on 128 x 256 tiles
@pytest.mark.parametrize("layout,M,n,K,chunks", [(0, 4096, 640, 8192, 3), (0, 4096, 384, 8192, 2), (0, 8192, 752, 16384, 2), (1, 4096, 8192, 384, 1),
                                                 (2, 640, 8192, 4096, 1), (0, 1672, 2880, 5720, 1), (0, 1400, 3704, 6184, 1), (0, 6672, 608, 4840, 1),
                                                 (1, 576, 10400, 6176, 1), (1, 320, 11920, 4672, 1), (1, 2473, 2712, 696, 1), (0, 237, 8296, 13120, 5),
                                                 (2, 1223, 1600, 12568, 6)])
def test_chunks_of_a_product(handle, layout, M, n, K, chunks):
    c = N.ntp_gemm_choice(layout, M, n, K, handle=handle)
    assert c["k_splits"] == chunks, c


def test_workspace_of_a_shard_of_three_heads_fits_the_static_scratch():
    """4096 tokens, hidden 8192: three chunks of the QKV projection."""
    assert N.ntp_workspace_bytes(Bd.NTP_CALL_ATTN_PROJ_SHARD, Bd.AttnShape(4096, 8192, 640, 384)) == 3 * 4096 * 640 * 4


SOURCE = r"""
#include <cstdio>
#include <initializer_list>
#include "ntp_internal.h"
// A handle on a device that is never reached: calls without operands stop at the first check behind the scratch size.
int main() {
  ntp_handle h;
  h.device = 0;
  static char scratch[256], out[16];
  h.static_scratch = scratch;
  int refused = 0, taken = 0;
  auto check = [&](const ntp_attn_shape_t& s, bool qkv, bool z) {
    int64_t need = 0;
    const ntp_attn_shape_t halves{s.M, s.H, qkv ? s.w_qkv : 0, z ? s.w_o : 0};
    // (the halves' forward products; the query covers the backward ones too, so it is asked per product)
    int64_t want = 0;
    for (const bool deep : {false, true}) {
      if (qkv && want < ntp::gemm_workspace_wish(&h, 0, s.M, s.w_qkv, s.w_qkv, s.H, deep)) want = ntp::gemm_workspace_wish(&h, 0, s.M, s.w_qkv, s.w_qkv, s.H, deep);
      if (z && want < ntp::gemm_workspace_wish(&h, 1, s.M, s.H, s.H, s.w_o, deep)) want = ntp::gemm_workspace_wish(&h, 1, s.M, s.H, s.H, s.w_o, deep);
    }
    if (ntp_workspace_bytes(&h, NTP_CALL_ATTN_PROJ_SHARD, &halves, &need) != NTP_OK || want > need) {
      printf("FAIL the query reports %lld bytes, the products use %lld\n", (long long)need, (long long)want);
      return false;
    }
    const int st = ntp_attn_proj_shard_fwd_static(&h, &s, nullptr, s.H, nullptr, s.H, qkv ? out : nullptr, s.w_qkv, nullptr, s.w_o, nullptr, s.H, z ? out : nullptr, s.H, nullptr);
    const int expected = want > int64_t(NTP_STATIC_SCRATCH_BYTES) ? NTP_ERR_SCRATCH_TOO_SMALL : NTP_ERR_INVALID_ARG;
    (want > int64_t(NTP_STATIC_SCRATCH_BYTES) ? refused : taken)++;
    if (st != expected) printf("FAIL %lld x %lld, w_qkv %lld, w_o %lld: %lld bytes, status %d\n", (long long)s.M, (long long)s.H, (long long)s.w_qkv, (long long)s.w_o, (long long)want, st);
    return st == expected;
  };
  for (int64_t M : {512, 1000, 2048, 4096, 4100, 8192})
    for (int64_t H : {1024, 2744, 5376, 8192, 11904, 16384})
      for (int64_t w = 128; w <= 4096; w += 8 * 13)
        if (!check({M, H, w, w}, true, false) || !check({M, H, w, w}, false, true) || !check({M, H, w, 256}, true, true)) return 1;
  printf("OK %d %d\n", refused, taken);
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_static_scratch_refuses_what_the_launches_could_use_more_room_for(tmp_path):
    src, exe = tmp_path / "static.cpp", str(tmp_path / "static")
    src.write_text(SOURCE)
    Bd.lib()  # (built)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, str(src), build.LIB_PATH, "-o", exe,
                    f"-Wl,-rpath,{build.HERE}", "-Wl,--allow-shlib-undefined"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    tag, refused, taken = res.stdout.split()
    assert tag == "OK" and int(refused) > 20 and int(taken) > 1000, res.stdout
