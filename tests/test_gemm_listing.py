"""What the compiled GEMM kernels have to hold, read from the compiler's listing.

The fp32 kernels read whole chunks of K with 16-byte loads at any alignment.
The few-row kernel waits for a chunk's activation copies (buffer_load ... lds) by
counting the weight loads issued after them, so in every block of its code the
copies have to come first.  Other instruction schedulers of the same compiler
take other orders wherever the source leaves them free; the source has to fix
this one for all of them.
"""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2609_01068_amd import build

SCHEDULERS = {"default": [], "iterative ILP": ["-mllvm", "-misched=gcn-iterative-ilp"],
              "no load clusters": ["-mllvm", "-misched-cluster=false"]}


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    folder = tmp_path_factory.mktemp("gemm")

    def compile_one(item):
        name, options = item
        out = str(folder / (name.replace(" ", "_") + ".s"))
        cmd = [build.hipcc()] + build._flags(False) + options + [
            "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm.hip"), "-o", out]
        subprocess.run(cmd, check=True, capture_output=True, text=True)
        with open(out) as f:
            return name, f.read()

    with cf.ThreadPoolExecutor(len(SCHEDULERS)) as ex:
        return dict(ex.map(compile_one, SCHEDULERS.items()))


@pytest.mark.parametrize("scheduler", SCHEDULERS)
def test_weight_loads_stay_behind_the_copies(listings, scheduler):
    kernels = re.findall(r"^(_ZN7outlets\S*gemm_stream\S*):[^\n]*\n(.*?)\.end_amdhsa_kernel", listings[scheduler],
                         re.M | re.S)
    assert kernels
    wrong = []
    for name, body in kernels:
        copies = loads = early = 0
        for line in body.split("\n"):
            if re.search(r"s_barrier|^\.LBB|s_cbranch|s_branch", line):
                loads = 0
            elif re.search(r"(global|flat)_load_dwordx4", line):
                loads += 1
            elif re.search(r"buffer_load_dwordx4.* lds", line):
                copies += 1
                early += loads > 0
        assert copies, name
        if early:
            wrong.append(name)
    assert not wrong, f"{len(wrong)} of {len(kernels)} kernels load weights before a copy"


def test_unaligned_fp32_rows_use_wide_loads(listings):
    """Loaded element by element, unaligned rows took twice as long as in
    16-byte pieces (d = 1,002, 6,000-27,000 tokens)."""
    kernels = re.findall(r"^(_ZN7outlets\S*gemm_f32_mfmaILi\d+ELb0E\S*):[^\n]*\n(.*?)\.end_amdhsa_kernel",
                         listings["default"], re.M | re.S)
    assert kernels
    for name, body in kernels:
        assert "global_load_dwordx4" in body, name


def _epilogues(listing, kernel):
    kernels = re.findall(r"^(_ZN7outlets\S*%s\S*):[^\n]*\n(.*?)\.end_amdhsa_kernel" % kernel, listing, re.M | re.S)
    assert kernels
    return [(name, body[body.rfind("v_mfma"):] if "v_mfma" in body else body) for name, body in kernels]


def test_rope_epilogue_reads_the_tables_once_per_tile(listings):
    """A row's position, slot and page are a chain of dependent loads; read
    by every lane for each of its 32 rows, they took 4% of a large prefill's
    q|k|v."""
    for name, epilogue in _epilogues(listings["default"], "gemm_mfma_256x256ILi6E"):
        assert len(re.findall(r"global_load_dword\s", epilogue)) <= 8, name


def test_scattered_value_stores_take_neighbouring_channels(listings):
    """Values of scattered rows leave two bytes at a time; with a lane's own
    channels in turn, each store touches 2 to 4 times the lines (12,288 x
    1,024 q|k|v of 512 decode rows: 66 us against 52)."""
    for kernel in ("gemm_mfma_256x256ILi6E", "splitk_reduce_qkv_rope"):
        for name, epilogue in _epilogues(listings["default"], kernel):
            assert "ds_bpermute" in epilogue, name
