"""The assembly of the GEMM kernels whose LDS reads are inline assembly (no GPU): the ping-pong kernel, persistent and with one workgroup per unit of work, and the
deep-pipelined one, alone and in shared launches; and the ring kernel's prefetch.  The compiler takes such a read's registers as written at once; that nothing touches them before the wait
is kept by the source's order, and checked in what the compiler makes of it, for every instantiation."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2504_06095_amd import build

from tests.test_host_attn_schedule import _code, _in_flight_faults, _symbols, _without_waits

# file, kernel, instantiations: seven tile shapes by epilogue; the 256 x 256 weight gradient with one workgroup per tile accumulates too
KERNELS = [("ntp_gemm_pp_nt", "gemm_pp_kernel", 21), ("ntp_gemm_pp_nn", "gemm_pp_kernel", 7), ("ntp_gemm_pp_tn", "gemm_pp_kernel", 14),
           ("ntp_gemm_nt", "gemm_pp_kernel", 7), ("ntp_gemm_nn", "gemm_pp_kernel", 7), ("ntp_gemm_tn", "gemm_pp_kernel", 8),
           ("ntp_gemm_deep", "gemm_deep_kernel", 32), ("ntp_gemm_deep", "gemm_deep_group_kernel", 2)]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm")

    def compile_one(name):
        s = str(out / f"{name}.s")
        build._run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.HIP_FLAGS, "-S", "--offload-device-only", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, os.path.join(build.CSRC, f"{name}.hip"), "-o", s])
        return name, open(s).read().splitlines()

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 8)) as pool:
        return dict(pool.map(compile_one, sorted({k[0] for k in KERNELS})))


@pytest.mark.parametrize("source,kernel,instantiations", KERNELS)
def test_registers_are_left_alone_while_reads_are_in_flight(assembly, source, kernel, instantiations):
    lines = assembly[source]
    starts = _symbols(lines, kernel)
    assert len(starts) == instantiations, [lines[s] for s in starts]
    for start in starts:
        code, labels = _code(lines, start)
        assert sum(op.startswith("v_mfma") for op, _, _ in code) >= 16 and sum(op.startswith("ds_read") for op, _, _ in code) >= 12
        assert not any("scratch_" in text for _, _, text in code), lines[start]
        faults = _in_flight_faults(code, labels)
        assert not faults, (lines[start], list(faults.values())[:5])
    # (the check sees a missing wait: the code in a straight line from the first read to the matrix instruction behind it)
    first = next(i for i, c in enumerate(code) if c[0].startswith("ds_read"))
    stop = next(i for i, c in enumerate(code) if i > first and c[0].startswith("v_mfma"))
    line = [c for c in code[first:stop + 1] if not c[0].startswith(("s_branch", "s_cbranch"))] + [("s_endpgm", [], "s_endpgm")]
    assert _in_flight_faults(_without_waits(line), {})


@pytest.mark.parametrize("source", ["ntp_gemm_nt", "ntp_gemm_nn", "ntp_gemm_tn"])
def test_prefetched_words_register_is_theirs_alone(assembly, source):
    """The ring kernel's prefetch to L2 loads words that nobody reads, in assembly: one register, which nothing else touches once a load may be in flight."""
    prefetching = 0
    for start in _symbols(assembly[source], "gemm_ring_kernel"):
        code, _ = _code(assembly[source], start)
        loads = [i for i, c in enumerate(code) if re.fullmatch(r"global_load_dword v\d+, v\d+, s\[\d+:\d+\]", c[2])]
        if not loads:
            continue
        prefetching += 1
        sinks = {code[i][1][0] for i in loads}
        assert len(sinks) == 1, assembly[source][start]
        touched = [c[2] for i, c in enumerate(code) if i not in loads and any(o & next(iter(sinks)) for o in c[1])]
        assert len(touched) == 1 and re.fullmatch(r"v_mov_b32_e32 v\d+, 0", touched[0]), (assembly[source][start], touched[:5])
    assert prefetching >= 8
