"""The host rules that choose a kernel form by sizes, compiled for the host and asked directly."""
import ctypes
import os
import subprocess

import pytest

from paper_2310_01801_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "paper_2310_01801_amd/csrc/fg_internal.h"
extern "C" int unit_threads(const fg_config* c) { return fg_unit_threads(*c); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    out = tmp_path_factory.mktemp("rules")
    (out / "rules.cpp").write_text(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", ROOT,
                    "-I", os.path.join(rocm, "include"), str(out / "rules.cpp"), "-o", str(out / "rules.so")], check=True)
    return ctypes.CDLL(str(out / "rules.so"))


def _cfg(U, n, S, d=64, dtype=binding.torch.bfloat16, **kw):
    return binding.make_config(U, 1, d, dtype, n, S, 0.95, 0.3, 0.3, **kw)


# A launch of the decode step holds fewer than 2^32 threads in one grid dimension. Short prompts with
# room for many generated tokens in a small pool reach 2^23 units within a card's memory.
@pytest.mark.parametrize("G", [1, 2, 8])
@pytest.mark.parametrize("n,S", [(8, 24), (16, 2032), (16, 2033), (16, 4000), (16, 8000)])
def test_decode_step_grid_stays_below_2_to_32_threads(rules, n, S, G):
    for U in (1 << 22, (1 << 22) + 1, (1 << 23) - 1, 1 << 23, (1 << 24) - 1):
        cfg = _cfg(U, n, S, cache_tokens=U * 8, group_size=G)
        assert binding.fastgen_workspace_bytes(cfg) > 0
        assert U * rules.unit_threads(ctypes.byref(cfg)) < 1 << 32, (U, n, S, G)
