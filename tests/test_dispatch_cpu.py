"""The host rules that choose a kernel form by sizes, compiled for the host and asked directly."""
import ctypes
import os
import struct
import subprocess

import msgpack
import pytest

from paper_2310_01801_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = """
#include "paper_2310_01801_amd/csrc/fg_internal.h"
extern "C" int unit_threads(const fg_config* c) { return fg_unit_threads(*c); }
extern "C" int sweep_form(int d, int pass, int U, int n, int G) { return fg_sweep_form_of(d, pass, U, n, G); }
extern "C" int once_form(int d, int U, int n, int G) { const fg_once_form f = fg_once_of(d, U, n, G); return f.waves * 100 + f.parts; }
extern "C" int once_f32_parts(int U, int n, int G) { return fg_once_f32_parts(U, n, G); }
extern "C" int once_long_parts(int d, int U, int n, int G) { return fg_once_long_parts(d, U, n, G); }
extern "C" int update_threads(const fg_config* c) { return fg_update_threads(*c); }
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


def _kernel_metadata(path):
    """Name -> metadata of every kernel in the AMDGPU code objects inside a library built here."""
    data, out, at = open(path, "rb").read(), {}, 0
    while (at := data.find(b"\x7fELF", at + 1)) > 0:
        if struct.unpack_from("<H", data, at + 18)[0] != 224:   # EM_AMDGPU
            continue
        phoff, (phentsize, phnum) = struct.unpack_from("<Q", data, at + 32)[0], struct.unpack_from("<HH", data, at + 54)
        for i in range(phnum):
            kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", data, at + phoff + i * phentsize)
            note, end = at + offset, at + offset + size
            while kind == 4 and note < end:   # PT_NOTE
                name_size, desc_size, note_type = struct.unpack_from("<III", data, note)
                desc = note + 12 + (name_size + 3) // 4 * 4
                if note_type == 32 and data[note + 12:note + 18] == b"AMDGPU":
                    out.update({k[".name"]: k for k in msgpack.unpackb(data[desc:desc + desc_size])["amdhsa.kernels"]})
                note = desc + (desc_size + 3) // 4 * 4
    return out


# Two workgroups of 512 threads of the update kernel stay on a CU: at most 128 vector registers each
# (512 per SIMD lane, four waves on it). The grouped one took 134.
def test_update_kernels_keep_two_workgroups_per_cu():
    kernels = {k: v for k, v in _kernel_metadata(binding.LIB_PATH).items() if "fg_decode_finish_kernel" in k}
    assert len(kernels) >= 8
    for name, meta in kernels.items():
        assert meta[".vgpr_count"] <= 128 and meta.get(".vgpr_spill_count", 0) == 0, (name, meta[".vgpr_count"])


def test_update_threads(rules):
    for U, n, S, G, want in ((512, 300, 16, 16, 512), (513, 300, 16, 16, 256), (513, 3072, 0, 9, 256), (513, 3072, 1, 9, 512),
                             (4096, 300, 16, 1, 512)):
        assert rules.update_threads(ctypes.byref(_cfg(U, n, S, group_size=G))) == want


# Forms of the bf16 sweeps at shapes whose times were far apart (first, second sweep): a few long units,
# which the split stream made slower; grouped short ones; blocks taken singly that fill the card as pairs
SPLIT_32, SPLIT_64, BLOCKS, PAIRS = range(4)


@pytest.mark.parametrize("d,U,n,G,want", [
    (128, 1, 1000, 1, (SPLIT_32, SPLIT_32)), (128, 1, 4096, 1, (SPLIT_64, SPLIT_64)), (128, 1, 8192, 1, (SPLIT_64, SPLIT_64)),
    (128, 1, 16384, 1, (PAIRS, PAIRS)), (128, 2, 16384, 1, (PAIRS, PAIRS)), (128, 1, 32768, 1, (PAIRS, PAIRS)),
    (64, 1, 32768, 1, (PAIRS, PAIRS)), (128, 8, 8192, 1, (SPLIT_64, SPLIT_64)), (128, 9, 7197, 8, (PAIRS, PAIRS)),
    (128, 2, 4096, 4, (SPLIT_64, SPLIT_64)), (128, 200, 230, 8, (PAIRS, PAIRS)), (128, 256, 300, 2, (PAIRS, PAIRS)),
    (128, 600, 128, 2, (PAIRS, PAIRS)), (64, 600, 128, 2, (PAIRS, BLOCKS)), (64, 256, 250, 4, (PAIRS, BLOCKS)),
    (64, 128, 1000, 1, (PAIRS, BLOCKS)), (128, 192, 1000, 1, (PAIRS, PAIRS)), (128, 160, 900, 1, (BLOCKS, PAIRS)),
    (128, 32, 333, 1, (SPLIT_64, SPLIT_64)), (128, 32, 2048, 1, (SPLIT_64, SPLIT_64)), (128, 1024, 2048, 1, (PAIRS, PAIRS)),
    (128, 4096, 1024, 1, (PAIRS, PAIRS)), (64, 432, 1337, 1, (PAIRS, PAIRS)),
])
def test_sweep_forms(rules, d, U, n, G, want):
    assert tuple(rules.sweep_form(d, p, U, n, G) for p in (1, 2)) == want


def test_every_accepted_size_has_a_sweep_form(rules):
    for d in (64, 128):
        for n in (1, 31, 256, 257, 1000, 131072):
            for U in (1, 7, 8, 9, 1000, 1 << 24):
                for G in (1, 2, 16):
                    forms = [rules.sweep_form(d, p, U, n, G) for p in (1, 2)]
                    assert all(0 <= f <= PAIRS for f in forms) and not (d == 128 and forms[1] == BLOCKS)
                    if U >= 1000 and n >= 256:
                        assert forms[0] == PAIRS, (d, n, U, G)


# The shapes of the two-sweep tests on the GPU do not go in one pass, and reach every form
def test_forms_of_the_tested_two_sweep_shapes(rules):
    seen = set()
    for d, U, n, G, want in ((64, 2, 1033, 1, (SPLIT_32, SPLIT_32)), (128, 1, 1025, 1, (SPLIT_32, SPLIT_32)), (128, 16, 1100, 1, (SPLIT_64, SPLIT_64)),
                             (64, 16, 1100, 1, (SPLIT_64, SPLIT_64)), (64, 9, 2049, 1, (SPLIT_64, SPLIT_64)), (128, 100, 1032, 1, (BLOCKS, PAIRS)),
                             (64, 100, 1032, 1, (BLOCKS, BLOCKS)), (64, 120, 1513, 1, (BLOCKS, BLOCKS)), (128, 50, 1513, 2, (BLOCKS, SPLIT_64)),
                             (128, 200, 1100, 1, (PAIRS, PAIRS)), (128, 4, 300, 8, (SPLIT_64, SPLIT_32)), (64, 8, 333, 2, (SPLIT_32, SPLIT_32)),
                             (64, 256, 64, 8, (PAIRS, SPLIT_64)), (64, 549, 78, 16, (PAIRS, BLOCKS)), (128, 600, 30, 16, (PAIRS, PAIRS)),
                             (64, 32, 256, 8, (BLOCKS, SPLIT_32)), (64, 4, 1100, 4, (SPLIT_64, SPLIT_32)), (64, 4, 1500, 1, (SPLIT_32, SPLIT_32)), (64, 260, 1029, 1, (PAIRS, PAIRS))):
        assert rules.once_form(d, U, n, G) == 1, (d, U, n, G)
        assert tuple(rules.sweep_form(d, p, U, n, G) for p in (1, 2)) == want, (d, U, n, G)
        seen |= {(d, p, form) for p, form in enumerate(want)}
    assert len(seen) == 15   # all but the single blocks of the second sweep at d = 128


F32, BF16 = binding.torch.float32, binding.torch.bfloat16


PART_SUMS = 64 << 20   # room for partial sums beside the static scratch


# Both float32 sweeps in one pass: at least two blocks of 16 rows per workgroup, partial sums within their room
def test_one_pass_f32_parts(rules):
    for n in (1, 63, 64, 200, 1000, 1024, 1025):
        for U in (1, 8, 32, 64, 200, 256, 300, 1000, 2048, 1 << 16, 1 << 22, (1 << 22) + 1, 1 << 24):
            for G in (1, 2, 16):
                parts = rules.once_f32_parts(U, n, G)
                if parts:
                    assert 64 <= n <= 1024 and U * parts >= 256 and (parts == 1 or parts <= n // 32) and (U + 7) * parts * 256 < 1 << 32
                assert parts < 2 or parts * U * n * 16 <= PART_SUMS, (U, n, G)
    for args, want in (((64, 1000, 1), 31), ((4, 128, 1), 0), ((16, 1000, 4), 31), ((300, 300, 1), 6), ((3000, 300, 1), 1), ((350, 1000, 8), 5)):
        assert rules.once_f32_parts(*args) == want, (args, rules.once_f32_parts(*args))


# Three to eight bf16 heads: one workgroup per unit wherever it holds the unit, but a few long ones (fewer and longer the
# more heads share the padded columns, and with full caches earlier)
def test_matrix_core_group_forms(rules):
    for U, tokens, G, dtype, forced, want in ((64, 3000, 8, BF16, -1, 512), (4, 4608, 8, BF16, -1, 512), (4, 3000, 4, BF16, -1, 0),
                                              (32, 3000, 3, BF16, -1, 0), (48, 3000, 3, BF16, -1, 512), (4, 1000, 4, BF16, 4, 512), (300, 2000, 4, BF16, 4, 512),
                                              (280, 3000, 3, BF16, 4, 0), (256, 4609, 4, BF16, -1, 0), (64, 3000, 9, BF16, -1, 0),
                                              (64, 3000, 2, BF16, -1, 0), (64, 3000, 8, F32, -1, 0),
                                              (8, 4506, 5, BF16, -1, 0), (1, 2822, 5, BF16, 3, 0), (24, 2706, 5, BF16, -1, 0), (4, 1600, 5, BF16, 3, 512),
                                              (64, 3200, 5, BF16, -1, 512), (7, 4264, 6, BF16, 3, 0), (24, 4000, 6, BF16, 3, 512), (8, 4575, 6, BF16, 4, 0),
                                              (1, 4600, 7, BF16, 4, 0), (1, 4600, 7, BF16, 3, 512), (4, 4600, 8, BF16, 4, 0), (11, 2085, 4, BF16, 4, 0),
                                              (24, 1600, 3, BF16, 4, 0), (96, 4000, 3, BF16, 4, 512), (2, 1819, 5, BF16, 2, 512), (4, 3974, 5, BF16, 2, 0),
                                              (7, 4590, 5, BF16, 0, 512)):
        assert rules.unit_threads(ctypes.byref(_cfg(U, tokens - 8, 8, 128, dtype, group_size=G, forced_policy=forced))) == want


def _profile_regions(U, n, G):
    return sum(-(-x // 256) * 256 for x in (U * G * n * 8, U * n * 8, U * n * 8, U * n, U * n * 4, U * 4, U * 40, U * 20, U * 4,
                                            (U + 1) * 8, U * 4, 32))


# Both bf16 sweeps in one pass: never longer than a workgroup's columns (512 with four waves), never more parts than
# blocks of 64 rows or more threads than a launch holds, the partial sums within their room, and not where the two
# sweeps were measured faster. 300 to 400 units of eight heads share theirs alike; 83 units in three parts each would
# put 33 workgroups on the 32 CUs of an XCD; above 512 units short prompts of few heads stay whole
def test_one_pass_profile(rules):
    for d in (64, 128):
        for G in (1, 2, 4, 8, 16):
            for n in (1, 64, 65, 128, 129, 512, 513, 1000, 1024, 1025, 131072):
                for U in (1, 8, 64, 128, 129, 256, 257, 300, 512, 1000, 2048, 2049, 1 << 22, (1 << 22) + 1, 1 << 24):
                    waves, parts = divmod(rules.once_form(d, U, n, G), 100)
                    assert waves in (0, 4, 8) and 1 <= parts <= -(-n // 64)
                    assert waves == 0 or (n <= 128 * waves and (U + 7) * parts * waves * 64 < 1 << 32)
                    assert not waves or parts == 1 or parts * U * n * 16 <= PART_SUMS, (d, U, n, G)
    for args, want in (((128, 4096, 1024, 1), 801), ((128, 4096, 512, 1), 401), ((128, 64, 1000, 1), 804), ((128, 32, 333, 1), 806),
                       ((128, 160, 400, 1), 403), ((128, 8, 1000, 1), 810), ((64, 1, 64, 1), 401), ((128, 64, 64, 4), 1), ((64, 256, 64, 8), 1),
                       ((64, 32, 256, 8), 1), ((64, 8, 333, 2), 1), ((128, 8, 512, 16), 1), ((64, 300, 1000, 8), 804), ((128, 1024, 2048, 1), 1),
                       ((128, 300, 1000, 8), 804), ((128, 350, 1000, 8), 802), ((128, 400, 1000, 8), 803), ((64, 83, 519, 16), 805),
                       ((64, 658, 159, 2), 401), ((64, 1746, 365, 1), 401), ((64, 1256, 183, 12), 401), ((64, 1099, 365, 16), 403)):
        assert rules.once_form(*args) == want, (args, rules.once_form(*args))


# The first 1024 columns of longer bf16 prompts in one pass: parts as above, at most the 17 blocks of the shortest such
# prompt and the room for their sums; few units of long prompts stay with the two sweeps, whose measured gain would be below 1
def test_first_columns_of_long_prompts(rules):
    for d in (64, 128):
        for n in (1, 1024, 1025, 1500, 2048, 3201, 5001, 8192, 8193, 131072):
            for U in (1, 8, 12, 95, 96, 179, 180, 1024, 4096, 1 << 22, (1 << 22) + 1):
                parts = rules.once_long_parts(d, U, n, 1)
                assert 0 <= parts <= 16 and (not parts or 1024 < n <= 8192)
                assert parts < 2 or parts * U * 1024 * 16 <= PART_SUMS
                assert (U + 7) * parts * 512 < 1 << 32
    for args, want in (((128, 1024, 2048), 2), ((128, 1024, 1337), 1), ((128, 1024, 4096), 3), ((128, 64, 1060), 4), ((128, 32, 2048), 8), ((128, 16, 2048), 16), ((64, 432, 1337), 1),
                       ((128, 640, 2048), 2), ((128, 150, 1060), 3), ((128, 32, 4096), 0), ((128, 100, 6000), 0), ((64, 4, 1060), 0), ((128, 8, 3000), 0)):
        assert rules.once_long_parts(*args, 1) == want, (args, rules.once_long_parts(*args, 1))


# Short prompts that the two sweeps were measured to serve faster, and their neighbours in one pass: up to 32 tokens with
# several heads, two blocks that are mostly empty, few units, a last round that stays mostly empty
def test_short_prompts_of_the_two_sweeps(rules):
    for args, want in (((128, 576, 22, 16), 0), ((128, 225, 21, 4), 0), ((128, 27, 10, 2), 0), ((64, 4151, 32, 2), 0), ((64, 3387, 21, 1), 0),
                       ((128, 482, 32, 4), 401), ((128, 1277, 16, 2), 401), ((128, 576, 33, 16), 401), ((64, 16, 77, 2), 0), ((64, 97, 95, 2), 402),
                       ((128, 40, 86, 2), 0), ((128, 54, 99, 2), 402), ((64, 549, 78, 16), 0), ((64, 2189, 66, 4), 0), ((64, 1398, 128, 4), 401),
                       ((64, 620, 139, 12), 0), ((64, 1161, 229, 6), 403), ((64, 2, 534, 4), 0), ((64, 3, 700, 4), 810), ((64, 1864, 537, 3), 0), ((64, 1219, 527, 8), 801), ((64, 2049, 1000, 1), 0),
                       ((64, 1447, 926, 1), 801), ((64, 459, 1002, 1), 801), ((128, 2049, 1000, 1), 801)):
        assert rules.once_form(*args) == (want or 1), (args, rules.once_form(*args))   # (1: no waves, one part)
    for args, want in (((130, 65, 4), 0), ((131, 71, 16), 0), ((114, 95, 8), 3), ((126, 118, 4), 4), ((83, 120, 16), 4), ((130, 65, 1), 2)):
        assert rules.once_f32_parts(*args) == want, (args, rules.once_f32_parts(*args))


# A context holds the partial sums whatever its cache pool, behind the regions of the profile; a usual pool's workspace
# (here d = 64, the smallest rows) holds them anyway
def test_workspace_holds_the_partial_sums(rules):
    for dtype, U, n, G in ((F32, 64, 1000, 1), (F32, 16, 1000, 4), (BF16, 64, 1000, 1), (BF16, 8, 1000, 1), (BF16, 1920, 1024, 1), (BF16, 300, 1000, 8)):
        parts = rules.once_f32_parts(U, n, G) if dtype is F32 else rules.once_form(64, U, n, G) % 100
        assert parts > 1
        least = _profile_regions(U, n, G) + parts * U * n * 16
        sizes = [binding.fastgen_workspace_bytes(_cfg(U, n, 0, 64, dtype, group_size=G, cache_tokens=pool)) for pool in (1, U * 8, U * n // 2, U * n, 0)]
        assert min(sizes) >= least and sizes == sorted(sizes), (U, n, G)
        pool = 2 * 64 * (4 if dtype is F32 else 2) * U * n
        assert pool >= parts * U * n * 16 and sizes[-1] >= _profile_regions(U, n, G) + pool


# Forms of the decode step at shapes whose times were far apart: nearly equal caches just above one unit per
# CU, long float32 rows, and their neighbours that gain from one workgroup per unit


@pytest.mark.parametrize("U,tokens,d,dtype,G,forced,want", [
    (257, 2600, 128, BF16, 1, 4, 0), (300, 4500, 128, BF16, 1, 4, 0), (300, 2000, 128, BF16, 2, 4, 0), (300, 1500, 128, F32, 1, 4, 0),
    (900, 4500, 128, BF16, 1, 3, 0), (300, 3600, 128, BF16, 1, -1, 512), (257, 1500, 128, BF16, 1, 4, 512), (257, 3000, 128, BF16, 1, 2, 512),
    (4, 2000, 128, BF16, 1, 4, 0), (32, 1000, 128, BF16, 1, 4, 0), (47, 1000, 128, F32, 2, 4, 0), (48, 1000, 128, BF16, 1, 4, 512),
    (4, 2000, 128, BF16, 1, 3, 512), (4, 2000, 128, BF16, 1, -1, 512), (32, 516, 128, F32, 1, 4, 512), (32, 500, 128, BF16, 1, 4, 512),
    (300, 4400, 128, BF16, 4, 4, 512), (500, 4500, 128, BF16, 1, 4, 512),
    (256, 4500, 128, BF16, 1, 4, 512), (400, 2600, 128, BF16, 1, 4, 512), (900, 3500, 128, BF16, 1, 3, 512),
    (400, 2500, 128, F32, 1, -1, 0), (640, 3500, 128, F32, 1, -1, 0), (400, 1800, 128, F32, 1, -1, 512), (400, 3500, 64, F32, 1, -1, 512),
    (256, 4400, 128, F32, 1, -1, 512), (1600, 4112, 128, BF16, 1, -1, 512), (640, 8320, 128, BF16, 1, -1, 0),
    (4096, 1280, 128, BF16, 1, -1, 256), (256, 2112, 128, BF16, 4, -1, 512), (32, 2048, 128, BF16, 1, -1, 512), (32, 2049, 128, BF16, 1, -1, 0),
])
def test_decode_step_forms(rules, U, tokens, d, dtype, G, forced, want):
    assert rules.unit_threads(ctypes.byref(_cfg(U, tokens - 8, 8, d, dtype, group_size=G, forced_policy=forced))) == want
