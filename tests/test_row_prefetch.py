"""The tile loops of the vote and of the exact assignment keep the next tile's
rows in flight while they compute the current one.  In the compiled kernels no
wait for vector memory stands between the row loads and the matrix products
that follow them: such a wait (a select on the loaded words was one) exposes
the whole latency of memory in every tile, which no result shows.  Partial
channel blocks (harmonic counts that are no multiple of 8), both dtypes.  And the
fp32 assignments that fill their registers do so without scratch memory, whose
set-up every launch would pay for.

Compiles six kernels with hipcc; runs without a GPU."""
import re
import shutil
import subprocess

import pytest

from paper_2609_16874_amd import build

VOTE = """template __global__ void k_vote_mfma<{T}, {F}, false, {fused}>(
    const {T} *__restrict__, int32_t, int32_t, const int32_t *__restrict__, const int32_t *__restrict__, int32_t,
    int32_t, int32_t, Tables, int32_t, int32_t, unsigned long long *__restrict__, cpe_centroid *__restrict__, int32_t,
    FusedArgs);"""
ASSIGN = """template __global__ void k_assign_mfma<{T}, {F}, {fast}>(
    const {T} *__restrict__, int32_t, int32_t, const int32_t *__restrict__, const int32_t *__restrict__, int32_t,
    int32_t, int32_t, double, Tables, const unsigned long long *__restrict__, unsigned long long *__restrict__,
    int32_t, int32_t, long long, int32_t, cpe_centroid *__restrict__, int32_t *__restrict__, int32_t *__restrict__,
    float *__restrict__, int32_t);"""
KERNELS = [VOTE.format(T="float", F=12, fused="false"), VOTE.format(T="_Float16", F=4, fused="true"),
           ASSIGN.format(T="_Float16", F=6, fast="false")]
FULL = [ASSIGN.format(T="float", F=5, fast="false"), ASSIGN.format(T="float", F=5, fast="true"),
        ASSIGN.format(T="float", F=8, fast="true")]


def waits_on_rows(body):
    """(products after row loads without a wait between, with one)."""
    free = waited = 0
    loads = wait = False
    for line in body.splitlines():
        if re.search(r"\bglobal_load_dwordx[24]\b", line):
            loads, wait = True, False
        elif loads and re.search(r"\bs_waitcnt\b.*vmcnt", line):
            wait = True
        elif loads and "v_mfma_f32_32x32x16_f16" in line:
            free, waited = free + (not wait), waited + wait
            loads = False
    return free, waited


def compiled(kernels, tmp_path):
    """The assembly of these instantiations."""
    src, out = tmp_path / "kernels.hip", tmp_path / "kernels.s"
    src.write_text('#include "k_mfma.hpp"\nnamespace cpe {\n' + "\n".join(kernels) + "\n}\n")
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-Wall")]
    subprocess.run(["hipcc", *flags, "-I", build.INCLUDE, "-I", build.CSRC, "-S", "--cuda-device-only", "-o", str(out),
                    str(src)], check=True, cwd=tmp_path, stderr=subprocess.DEVNULL)
    return out.read_text()


needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


@needs_hipcc
def test_no_wait_between_row_loads_and_products(tmp_path):
    bodies = re.findall(r"^(_Z\w*(?:k_vote_mfma|k_assign_mfma)\w*):.*?\n(.*?)\n\s*s_endpgm\b.*?\.Lfunc_end",
                        compiled(KERNELS, tmp_path), flags=re.S | re.M)
    assert len(bodies) == len(KERNELS)
    for name, body in bodies:
        free, waited = waits_on_rows(body)
        assert free >= 1 and waited == 0, (name, free, waited)


@needs_hipcc
def test_full_kernels_need_no_scratch(tmp_path):
    sizes = re.findall(r"\.name:\s+(_Z\w*k_assign_mfma\w*)\n\s+\.private_segment_fixed_size: (\d+)",
                       compiled(FULL, tmp_path))
    assert len(sizes) == len(FULL)
    assert all(int(n) == 0 for _, n in sizes), sizes
