"""Shapes at the edges of the kernels' tiles and dispatch rules, against the float64 oracle."""
import math

import pytest
import torch

import fg_harness as H
from paper_2310_01801_amd import binding, synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS


def _compare(name, n, S, d, dtype, heads, G=1, probe_steps=(), forced=-1, **kw):
    w = W["llama7b_b1"].scaled(name=name, layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=d,
                               dtype=dtype, seed=900 + n, **kw)
    run = H.GpuRun(w, range(w.num_units), group_size=G, forced_policy=forced)
    rep = H.compare(run, probe_steps=probe_steps)
    H.log_report(f"{name} n={n} S={S} d={d} {dtype} G={G}", rep)
    return rep


# float32 sweeps: tiles of 16, four waves that take the tiles in turn (17 = one full tile and one
# row, 65 = a fifth tile that starts the second turn), and a unit count that is no multiple of 8
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 129, 300])
@pytest.mark.parametrize("d,G", [(64, 1), (128, 1), (128, 2)])
def test_f32_sweeps_at_tile_edges(n, d, G):
    rep = _compare("f32_edges", n, 2, d, "f32", 5, G)
    # float64 sums, (m, 1/l) held as floats: half an ulp (6e-8) per row, far below it in the mean
    assert rep.max_recovery_err < 6e-8


# the decode step's two forms: one workgroup per unit (256 or 512 threads; units ordered by size in
# one launch up to 1024 of them, in two up to 16384, unordered above) or split-KV. Unit counts and
# lengths on both sides of every line; the oracle follows a few units at the ends and in the middle.
@pytest.mark.parametrize("heads,n,S,d,dtype", [
    (3, 1, 3, 128, "bf16"),        # a unit of one token
    (5, 33, 6, 64, "bf16"),        # one tile and one row of a wave (d = 64: 32 rows)
    (4, 65, 6, 64, "f32"),
    (4, 1020, 4, 128, "bf16"),     # half of, at and above 1 MiB per unit, fewer units than CUs
    (4, 2044, 4, 128, "bf16"),
    (4, 2045, 4, 128, "bf16"),
    (255, 40, 3, 128, "bf16"), (256, 40, 3, 128, "bf16"),
    (256, 4100, 2, 64, "bf16"),
    (256, 4606, 2, 64, "bf16"), (256, 4607, 2, 64, "bf16"),   # at and above the line to split-KV
    (1024, 24, 3, 64, "bf16"), (1025, 24, 3, 64, "f32"), (2047, 24, 3, 64, "bf16"), (2048, 24, 3, 64, "bf16"),
    (16384, 9, 2, 64, "bf16"), (16385, 9, 2, 64, "bf16"),
])
def test_decode_step_forms(heads, n, S, d, dtype):
    w = W["llama7b_b1"].scaled(name="forms", layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=d,
                               dtype=dtype, seed=700 + n)
    run = H.GpuRun(w, range(w.num_units))
    check = sorted({0, 1, 2, heads // 2, heads - 2, heads - 1} & set(range(heads)))
    rep = H.compare(run, check_units=check, cover_policies=1)
    H.log_report(f"decode forms U={heads} n={n} S={S} d={d} {dtype}", rep)


# steps that release several tokens at once: a frequent budget next to a window, many steps
@pytest.mark.parametrize("forced,r_f,r_l", [(3, 0.3, 0.1), (3, 0.05, 0.02), (2, 0.5, 0.3)])
def test_evictions_of_the_per_unit_step(forced, r_f, r_l):
    rep = _compare("evictions", 150, 40, 64, "bf16", 6, forced=forced, r_f=r_f, r_l=r_l, probe_steps=(7, 20))
    assert rep.policies == {forced: 6}


# policy selection: tokens in registers (1, 2, 4, 8 slots of 512 threads for few units, 2, 4, 8, 12 of
# 256 for many, 8 of 1024 for long prompts) or re-read: both sides of every line
@pytest.mark.parametrize("heads,n", [(3, 512), (3, 513), (3, 1024), (3, 1025), (2, 2049), (2, 4096), (2, 4097), (1, 8192),
                                     (1, 8193), (513, 512), (513, 513), (513, 1025), (513, 2049), (513, 3073)])
def test_selection_sizes(heads, n):
    w = W["llama7b_b1"].scaled(name="selection", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=64,
                               seed=800 + n)
    run = H.GpuRun(w, range(w.num_units))
    rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}))
    H.log_report(f"selection U={heads} n={n}", rep)


# bf16 prompts of all lengths around tiles and blocks, and local windows whose edge falls inside, at and across tiles.
# Most go in one pass; the forms of the two sweeps have the test after this one
@pytest.mark.parametrize("heads,n,d,G", [
    (2, 31, 128, 1), (2, 32, 64, 1), (3, 33, 128, 1), (3, 63, 64, 2), (3, 65, 128, 1), (5, 129, 128, 2), (4, 300, 128, 8),
    (24, 333, 128, 1), (24, 257, 64, 1), (200, 400, 128, 1), (200, 400, 64, 1), (9, 2049, 64, 1),
    (800, 255, 128, 1), (800, 257, 128, 1), (800, 513, 64, 1), (400, 400, 128, 2),
])
def test_bf16_sweep_forms(heads, n, d, G):
    for window in (1, 31, 33, max(1, n // 3)):
        w = W["llama7b_b1"].scaled(name="sweeps", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=d,
                                   r_l=min(1.0, (window + 0.5) / n), seed=600 + n)
        run = H.GpuRun(w, range(w.num_units), group_size=G)
        rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}))
        H.log_report(f"sweep forms U={heads} n={n} d={d} G={G} w={window}", rep)


# bf16 sweeps: the split stream with one or two fragments of 32 owners (few units), 256-owner blocks taken singly (first
# sweep; both at d = 64) or in pairs, by unit count: prompts above 1024 tokens, and the short ones of several heads that
# one pass does not serve (the form of every shape here is asserted in test_dispatch_cpu.py)
@pytest.mark.parametrize("heads,n,d,G", [
    (2, 1033, 64, 1), (1, 1025, 128, 1), (16, 1100, 128, 1), (16, 1100, 64, 1), (9, 2049, 64, 1), (100, 1032, 128, 1), (100, 1032, 64, 1),
    (120, 1513, 64, 1), (50, 1513, 128, 2), (200, 1100, 128, 1), (4, 300, 128, 8), (8, 333, 64, 2), (256, 64, 64, 8), (549, 78, 64, 16),
    (600, 30, 128, 16), (32, 256, 64, 8), (260, 1029, 64, 1),
])
def test_two_sweep_forms(heads, n, d, G):
    for window in (1, 31, 33, max(1, n // 3)):
        w = W["llama7b_b1"].scaled(name="two_sweeps", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=d,
                                   r_l=min(1.0, (window + 0.5) / n), seed=600 + n)
        run = H.GpuRun(w, range(w.num_units), group_size=G)
        run.fg.fastgen_enable_timing(1)
        rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}))
        assert run.fg.fastgen_read_timing()["sweep2"][1] == 1
        H.log_report(f"two sweeps U={heads} n={n} d={d} G={G} w={window}", rep)


# Both float32 sweeps in one pass: tiles of 16, four waves that hold 4, 8 or 16 of them each (256, 512 and 1024 columns),
# one or several workgroups per unit, windows whose edge falls in, at and across tiles
@pytest.mark.parametrize("heads,n,d,G", [
    (128, 64, 64, 1), (128, 65, 128, 1), (64, 129, 64, 2), (64, 256, 128, 1), (64, 257, 64, 1), (40, 512, 128, 1), (40, 513, 64, 1),
    (16, 1000, 128, 1), (12, 1024, 64, 3), (300, 100, 128, 1), (2100, 70, 64, 1),
])
def test_f32_one_pass(heads, n, d, G):
    for window in (1, 16, 17, n // 3):
        w = W["llama7b_b1"].scaled(name="f32_one_pass", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=d, dtype="f32",
                                   r_l=min(1.0, (window + 0.5) / n), seed=700 + n)
        run = H.GpuRun(w, range(w.num_units), group_size=G)
        rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}))
        H.log_report(f"float32 one pass U={heads} n={n} d={d} G={G} w={window}", rep)


# The exponentials' shift starts at 0 and moves only for logits beyond 2^900: one such key early, late, and all of them
@pytest.mark.parametrize("pattern", ["early", "late", "all", "negative"])
def test_f32_one_pass_with_huge_logits(pattern):
    U, n, d = 16, 700, 128
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    Q, K = (torch.randn(U, n, d, generator=gen, device="cuda:0") for _ in range(2))
    Q[:, :, 0], K[:, :, 0] = 200.0, 0.0
    at = {"early": 3, "late": 650, "all": 40, "negative": 40}[pattern]
    K[:, at, 0] = 100.0                                     # 2^2551
    if pattern == "all":
        K[:, :, 0] += 90.0
    if pattern == "negative":
        K[:, :, 0] -= 170.0
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    cls[0, at] = 1
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.float32, n, 4, 0.95, 0.3, 0.3))
    _, recovery, _ = fg.fastgen_profile(Q, K, cls)
    fg.close()
    assert float((recovery[:, 0].cpu() - (n - at) / n).abs().max()) < 1e-6   # rows from `at` on give it all their mass


# The form of the pass follows from the shape alone: a pool that holds all, some or none of the partial sums of workgroups
# that share a unit gives the same bits, and so does the entry point without a context
@pytest.mark.parametrize("U,n,d,G,dtype", [(16, 700, 128, 1, torch.float32), (64, 1000, 64, 1, torch.float32), (16, 1000, 64, 1, torch.bfloat16),
                                           (32, 333, 128, 1, torch.bfloat16), (64, 400, 128, 4, torch.bfloat16), (640, 1000, 64, 1, torch.bfloat16)])
def test_one_pass_with_any_pool(U, n, d, G, dtype):
    gen = torch.Generator(device="cuda:0").manual_seed(4)
    Q, K = (torch.randn(x, n, d, generator=gen, device="cuda:0", dtype=dtype) for x in (U * G, U))
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    cls[0, 0] = 1
    cfg = binding.make_config(U, 1, d, dtype, n, 4, 0.95, 0.3, 0.3, group_size=G)
    want = (torch.empty(U, dtype=torch.int32, device="cuda:0"), torch.empty((U, 5), dtype=torch.float64, device="cuda:0"),
            torch.empty((U, 5), dtype=torch.int32, device="cuda:0"))
    binding.fastgen_profile_static(cfg, Q, K, cls, *want)
    for pool in (0, U * 8, U * n * 2 // 5):
        cfg.cache_tokens = pool
        fg = binding.FastGen(cfg)
        fg.workspace.fill_(255)
        fg.fastgen_enable_timing(1)
        got = fg.fastgen_profile(Q, K, cls)
        torch.cuda.synchronize()
        assert fg.fastgen_read_timing()["sweep2"][1] == 0
        assert all(torch.equal(x, y) for x, y in zip(got, want)), pool
        fg.close()


# In a small pool the partial sums lie over everything behind the profile's regions, the step's scratch included: what
# follows reads none of it
@pytest.mark.parametrize("U,n,d,G,dtype,forced", [(16, 1000, 64, 1, torch.float32, 0), (16, 1000, 64, 1, torch.bfloat16, 2), (64, 400, 128, 4, torch.bfloat16, 0),
                                                  (24, 900, 64, 9, torch.float32, 2)])
def test_session_in_a_small_pool_after_one_pass(U, n, d, G, dtype, forced):
    gen = torch.Generator(device="cuda:0").manual_seed(6)
    Q, K, V = (torch.randn(x, n, d, generator=gen, device="cuda:0", dtype=dtype) for x in (U * G, U, U))
    q, k, v = (torch.randn(3, x, d, generator=gen, device="cuda:0", dtype=dtype) for x in (U * G, U, U))
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    cls[0, :3] = 1
    seen = []
    for pool in (0, U * 64):
        cfg = binding.make_config(U, 1, d, dtype, n, 3, 0.95, 0.03, 0.03, forced_policy=forced, cache_tokens=pool, group_size=G)
        fg = binding.FastGen(cfg)
        fg.workspace.fill_(255)
        fg.fastgen_profile(Q, K, cls)
        fg.fastgen_compact(K, V)
        outs = [fg.fastgen_decode_step(q[t], k[t], v[t], cls[:, 5].contiguous()) for t in range(2)]
        outs += fg.fastgen_decode_step_probe(q[2], k[2], v[2], cls[:, 5].contiguous())
        st = fg.fastgen_export_state(rows=True)
        assert int(st["status"].item()) == 0
        seen.append(outs + [st[x] for x in ("lengths", "positions", "scores", "keys", "values")])
        fg.close()
    assert all(torch.equal(x, y) for x, y in zip(*seen))


# Three to eight bf16 heads on the matrix cores: tiles of 32 tokens (two sets of 16) over eight waves, four and eight
# columns, prompts of which some waves have no tile, longest units, every policy, probed steps
@pytest.mark.parametrize("heads,n,S,d,G,forced", [
    (3, 1, 3, 128, 3, -1), (3, 15, 4, 64, 4, 2), (3, 16, 4, 128, 4, 3), (3, 31, 4, 128, 8, 2), (3, 32, 4, 64, 5, 3), (5, 33, 40, 128, 4, -1),
    (5, 255, 4, 128, 3, 2), (5, 257, 12, 64, 8, -1), (40, 480, 6, 128, 6, -1), (33, 2300, 4, 128, 4, 3), (3, 4600, 8, 64, 7, -1),
    (5, 700, 6, 128, 8, 4), (5, 700, 6, 64, 4, 1), (257, 300, 4, 128, 4, -1),
])
def test_matrix_core_group_steps(heads, n, S, d, G, forced):
    w = W["llama7b_b1"].scaled(name="group_mfma", layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=d,
                               dtype="bf16", seed=1100 + n)
    run = H.GpuRun(w, range(w.num_units), group_size=G, forced_policy=forced)
    rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}), probe_steps=(1, 2))
    H.log_report(f"matrix-core group U={heads} n={n} S={S} d={d} G={G} forced={forced}", rep)


# A head whose keys outgrow each other from tile to tile moves its shift in every one of them; weights of 2^-200 and
# less beside it count nothing
def test_matrix_core_group_with_rising_logits():
    U, n, d, G = 8, 600, 128, 4
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    Q, K, V = (torch.randn(x, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for x in (U * G, U, U))
    K[:, :, 0] = torch.arange(n, device="cuda:0", dtype=torch.bfloat16) * 0.25
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 2, 0.95, 0.3, 0.3, forced_policy=4, group_size=G))
    fg.fastgen_profile(Q, K, cls)
    fg.fastgen_compact(K, V)
    q, k, v = (torch.randn(x, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for x in (U * G, U, U))
    q[:, 0] = torch.tensor([0.0, 4.0, 16.0, -16.0], device="cuda:0", dtype=torch.bfloat16).repeat(U)
    out = fg.fastgen_decode_step(q, k, v, torch.zeros(1, dtype=torch.uint8, device="cuda:0")).float().view(U, G, d)
    fg.close()
    Kf, Vf = torch.cat([K, k[:, None]], 1).double().cpu(), torch.cat([V, v[:, None]], 1).double().cpu()
    a = torch.softmax(q.view(U, G, d).double().cpu() @ Kf.transpose(1, 2) / d ** 0.5, dim=2)
    assert float((out.cpu().double() - a @ Vf).abs().max()) < 2e-2   # half a bf16 step below 8 is 2^-6


# The scores of such heads: every tile keeps its exponentials under the shift of its wave at that moment, the sums are
# rescaled whenever the shift moves, and the factors of the tiles meet at the end. Logits that rise and fall by half a
# power of two per token (the shift moves in every tile, or once), and by 32 of them (factors of 2^-4096 and less).
# Ratios of 1 keep every token, so that the scores grow by the step's attention and the probe sees whole classes. Logits
# of up to 2e4 powers of two in float64: 2e4 x 2^-53 each, some of them added.
@pytest.mark.parametrize("d,G", [(128, 4), (64, 4), (128, 8), (64, 8), (128, 3), (64, 6)])
@pytest.mark.parametrize("forced", [2, 3])
@pytest.mark.parametrize("slope", [0.25, -0.25, 16.0, -16.0])
def test_matrix_core_group_scores_with_moving_shifts(d, G, forced, slope):
    U, n = 6, 611
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    Q, K, V = (torch.randn(x, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for x in (U * G, U, U))
    ramp = torch.arange(n + 1, device="cuda:0") * abs(slope)
    ramp = (ramp if slope > 0 else ramp.flip(0)).bfloat16()
    K[:, :, 0] = ramp[:n]
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    cls[0, ::7], cls[0, 3::11] = 1, 2
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 2, 0.95, 1.0, 1.0, forced_policy=forced, group_size=G))
    fg.fastgen_profile(Q, K, cls)
    fg.fastgen_compact(K, V)
    before = fg.fastgen_export_state()["scores"].view(U, n)
    q, k, v = (torch.randn(x, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for x in (U * G, U, U))
    k[:, 0] = ramp[n]
    q[:, 0] = torch.tensor([0.0, 4.0, 16.0, -16.0, 8.0, -8.0, 1.0, -2.0], device="cuda:0", dtype=torch.bfloat16)[:G].repeat(U)
    new_class = torch.ones(1, dtype=torch.uint8, device="cuda:0")
    out, probe = fg.fastgen_decode_step_probe(q, k, v, new_class)
    after = fg.fastgen_export_state()["scores"].view(U, n + 1)
    fg.close()
    Kd, Vd = torch.cat([K, k[:, None]], 1).double().cpu(), torch.cat([V, v[:, None]], 1).double().cpu()
    scale = float(torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32))
    a = torch.softmax(q.view(U, G, d).double().cpu() @ Kd.transpose(1, 2).contiguous() * scale, dim=2)
    gained = after - torch.cat([before, torch.zeros_like(before[:, :1])], 1)
    assert float((gained.cpu() - a.sum(1)).abs().max()) < 1e-10
    held = torch.cat([cls[0], new_class]).cpu()
    masses = [(a.mean(1) * ((held & bits) != 0)).sum(1) for bits in (1, 3)] + [torch.ones(U, dtype=torch.float64)] * 3
    assert float((probe.cpu() - torch.stack(masses, 1)).abs().max()) < 1e-10
    assert float((out.float().view(U, G, d).cpu().double() - a @ Vd).abs().max()) < 2e-2   # half a bf16 step below 8 is 2^-6


# Both bf16 sweeps in one pass: fragments of 32 columns, blocks of 64 rows, four and eight waves, prompt lengths
# around each and around a wave's next fragment (128, 256), windows whose edge falls in the first, the second or both
# row fragments of a block; one and several workgroups per unit, even and odd numbers of blocks for them; grouped
# heads go through the columns anew one after the other
@pytest.mark.parametrize("heads,n,d,G", [
    (64, 1, 128, 1), (1, 31, 128, 1), (128, 33, 64, 1), (4, 63, 128, 1), (64, 65, 128, 1), (192, 97, 128, 2), (64, 129, 128, 1),
    (192, 130, 64, 3), (300, 257, 64, 1), (300, 385, 128, 1), (300, 511, 128, 2), (513, 512, 64, 1), (64, 513, 128, 1), (192, 700, 64, 2),
    (128, 993, 64, 1), (3, 1023, 128, 1), (257, 1024, 128, 1), (20, 960, 64, 5), (2100, 130, 64, 1),
])
def test_bf16_one_pass(heads, n, d, G):
    for window in (1, 30, 64, 97, n):
        w = W["llama7b_b1"].scaled(name="one_pass", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=d,
                                   r_l=min(1.0, (window + 0.5) / n), seed=900 + n)
        run = H.GpuRun(w, range(w.num_units), group_size=G)
        rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}))
        H.log_report(f"one pass U={heads} n={n} d={d} G={G} w={window}", rep)


# Prompts of one block: a wave per tile of 32 rows and columns, the second row of tiles empty, partly filled and full;
# one to sixteen heads after one another; windows inside, at the edge of and beyond a tile
@pytest.mark.parametrize("heads,n,d,G", [
    (5, 1, 64, 1), (300, 17, 128, 1), (9, 32, 128, 1), (64, 33, 128, 2), (70, 50, 64, 2), (300, 63, 128, 5), (200, 64, 128, 3), (300, 64, 64, 1), (260, 64, 128, 16), (2000, 64, 64, 1),
])
def test_prompts_of_one_block(heads, n, d, G):
    for window in sorted({1, 2, 31, 32, 33, n // 2, n - 1, n} & set(range(1, n + 1))):
        w = W["llama7b_b1"].scaled(name="one_block", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=d,
                                   r_l=min(1.0, (window + 0.5) / n), seed=800 + n)
        run = H.GpuRun(w, range(w.num_units), group_size=G)
        rep = H.compare(run, check_units=sorted({0, heads // 2, heads - 1}))
        H.log_report(f"one block U={heads} n={n} d={d} G={G} w={window}", rep)


# The first 1024 columns of longer prompts in one pass, the triangle behind them in two sweeps that leave and take row
# sums: triangles of one row, of a tile and of a block more or less, one and several workgroups per unit, grouped heads,
# windows inside a block, up to the seam at column 1024 and beyond it
@pytest.mark.parametrize("heads,n,d,G", [
    (8, 1025, 128, 1), (16, 1056, 64, 1), (64, 1087, 128, 2), (300, 1088, 64, 1), (256, 1313, 128, 1), (13, 1500, 128, 4), (200, 2111, 64, 1),
])
def test_long_prompts_in_one_pass_and_two_sweeps(heads, n, d, G):
    for window in (1, 64, 1024, n - 30, n):
        w = W["llama7b_b1"].scaled(name="long_pass", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=d,
                                   r_l=min(1.0, (window + 0.5) / n), seed=700 + n)
        run = H.GpuRun(w, range(w.num_units), group_size=G)
        rep = H.compare(run, check_units=sorted({0, heads - 1}))
        H.log_report(f"long pass U={heads} n={n} d={d} G={G} w={window}", rep)


# Row masses of the one-pass form. A float32 normaliser is off by up to 2^-24, 2.5e-8 in the root mean square over its
# mantissas; with the rounding of a row's partial sums and of its probabilities, all without a preference, 3.5e-8 a row (40 runs of
# 21312 rows scatter by 2.4e-10, with running maxima as with shifts from the rows before). Over 16 runs of that size the mean
# is within 4 x 3.5e-8 / 584; over four it was not, for no fault. A shift that moves with every tile and a hardware
# exponential for every rescaling of it would show as 1e-9 and more.
@pytest.mark.parametrize("U,n,d", [(64, 333, 128), (300, 400, 64), (128, 1000, 64)])
def test_one_pass_row_masses_have_no_bias(U, n, d):
    masses = []
    for seed in range(16):
        gen = torch.Generator(device="cuda:0").manual_seed(seed)
        Q, K = (torch.randn(U, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
        cls = torch.ones((1, n), dtype=torch.uint8, device="cuda:0")
        fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 0.3, 0.3))
        _, recovery, _ = fg.fastgen_profile(Q, K, cls)
        masses.append(float(recovery[:, 0].mean()) - 1.0)
        fg.close()
    assert abs(sum(masses) / 16) < 2.3e-10, masses


# Logits far beyond what a float32 exponential holds without a shift: a key that outweighs all others by 2^600
# and more, first in the prompt, in a later block, and in the other wave's fragment.
@pytest.mark.parametrize("n,at", [(100, 0), (300, 170), (1000, 40)])
def test_one_pass_with_huge_logits(n, at):
    U, d = 256, 128
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    Q, K = (torch.randn(U, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
    Q[:, :, 0], K[:, :, 0], K[:, at, 0] = 64.0, 0.0, 120.0
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    cls[0, at] = 1
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 0.3, 0.3))
    policy, recovery, _ = fg.fastgen_profile(Q, K, cls)
    fg.close()
    want = (n - at) / n   # every row from `at` on gives the key all its mass, the rows before it give none
    assert float((recovery[:, 0].cpu() - want).abs().max()) < 1e-6


# A row's shift is what the row 64 before came to. Logits whose rows lie up to 130 powers of two higher or lower than that
# one, in the first and later blocks, in whole blocks, single rows and the last row, with one and several workgroups per
# unit and with heads after one another. All keys share the offset, so the probabilities keep the size of a plain
# prompt's; a dot product of up to 600 over eight rounded steps in float32 is good to 8 x 2^-24 x 600 / sqrt(d), so the masses to
# 3.6e-5 (d = 64). So these are of the ways that a block can take; what they cost in precision is tested with exact products below.
@pytest.mark.parametrize("U,n,d,G", [(2, 1, 128, 1), (300, 64, 128, 1), (300, 130, 64, 1), (256, 1200, 128, 1), (16, 1100, 64, 2), (20, 333, 128, 1), (300, 700, 128, 1), (64, 1000, 64, 1), (200, 500, 64, 2)])
@pytest.mark.parametrize("rows", ["high", "low", "alternate", "single", "last"])
def test_one_pass_with_rows_far_from_the_ones_before(U, n, d, G, rows):
    gen = torch.Generator(device="cuda:0").manual_seed(n + d)
    Q, K = (torch.randn(x, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for x in (U * G, U))
    i = torch.arange(n, device="cuda:0")
    step = {"high": 0 * i + 1, "low": 0 * i - 1, "alternate": torch.where((i // 40) % 2 == 0, 1, -1),
            "single": (i % 97 == 50).int() - (i % 89 == 70).int(), "last": (i == n - 1).int()}[rows]
    Q[:, :, 0], K[:, :, 0] = (step * 64).bfloat16(), 8.0
    cls = (i % 3 == 0).to(torch.uint8)[None].contiguous()
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 0.3, 0.3, group_size=G))
    _, recovery, _ = fg.fastgen_profile(Q, K, cls)
    fg.close()
    scale = float(torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32))
    some = sorted({0, U // 2, U - 1})
    x = Q.view(U, G, n, d)[some].double().cpu().matmul(K[some].double().cpu().transpose(1, 2).contiguous()[:, None]) * scale
    x = x.masked_fill(torch.ones(n, n).triu(1).bool(), -math.inf)
    want = torch.softmax(x, dim=3)[:, :, :, cls[0].cpu() != 0].sum(3).mean((1, 2))
    assert float((recovery[some, 0].cpu() - want).abs().max()) < 3.6e-5


# Rows that lie a given number of powers of two above the rows 64 before, with products that are exact in float32 (an offset
# per block of rows and a number per column), against float64 with the factor that the device takes. What is left
# is the rounding of the exponential's argument at its own size: within 8 where a row's maximum is its shift (logits within 4
# of their middle), uniformly 2^-22, 9.5e-8 of the value in the root mean square; within 16 where a sum of up to 2^14 is accepted, twice that;
# the hardware exponential, the normaliser and the sums add less than 5e-8. A column's relative error so stays
# below 1.1e-7 (redone) and 2e-7 (accepted) in the root mean square. Sums of up to 2^100, accepted, made 1.2e-7 to 3.5e-7.
@pytest.mark.parametrize("U,n,d", [(64, 1000, 128), (300, 1024, 64), (300, 500, 128), (64, 1500, 128), (300, 1100, 64)])
@pytest.mark.parametrize("step", [64, 24, 6, -6, -24, -64])
def test_one_pass_keeps_its_precision_where_rows_lie_apart(U, n, d, step):
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    Q, K = (torch.zeros(U, n, d, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
    c = torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32) * torch.tensor(math.log2(math.e), dtype=torch.float32)
    block = torch.arange(n, device="cuda:0") // 64
    Q[:, :, 0] = block.float() if step > 0 else block.max() - block.float()   # times K's: raw products of a step
    K[:, :, 0] = round(abs(step) / float(c))
    K[:, :, 1] = torch.randint(-120, 121, (U, n), generator=gen, device="cuda:0") / (4.0 if d == 128 else 8.0)
    Q[:, :, 1] = 1.0
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 1.0, 0.5, forced_policy=3))
    fg.fastgen_profile(Q, K, cls)
    fg.fastgen_compact(K, K)
    got = fg.fastgen_export_state()["scores"][:U * n].view(U, n).cpu()
    fg.close()
    x = torch.matmul(Q[:8].double().cpu(), K[:8].double().cpu().transpose(1, 2).contiguous()) * float(c) * math.log(2.0)
    want = torch.softmax(x.masked_fill(torch.ones(n, n).triu(1).bool(), -math.inf), dim=2).sum(1)
    error = ((got[:8] - want) / want).pow(2).mean().sqrt()
    print(f"rows {step} apart, U={U} n={n} d={d}: {float(error):.2e}")
    assert float(error) < (1.1e-7 if abs(step) > 10 else 2e-7)


# The rows' sums behind column 1024 reach the one pass with more than 24 bits: 1 + 2^-24 of the columns there (in tiles of
# their own), which 24 bits make 1 or 1 + 2^-23, and one column before them of a random weight A per unit. Column 1024 is the sum of 1 / (A + 1)
# over 64 rows and of 1 / (A + 1 + 2^-24) over 192. What is left is the rounding of the normalisers and of their sums, 4e-8 a unit
# at most in the root mean square and without a preference, four times that over 512 units 7e-9, and A's, whose hardware exponential counts
# for a fifth or less (1.3e-9 and 3.0e-9 measured); sums of 24 bits are 2.8e-8 and 3.6e-8 off.
@pytest.mark.parametrize("U,d", [(512, 64), (512, 128)])
def test_row_sums_behind_the_one_pass_keep_their_bits(U, d):
    n = 1280
    gen = torch.Generator(device="cuda:0").manual_seed(d)
    Q, K = (torch.zeros(U, n, d, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
    c = float(torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32) * torch.tensor(math.log2(math.e), dtype=torch.float32))
    Q[:, :, 0] = 1.0
    K[:, :, 0] = -300.0 / c
    K[:, 0, 0] = (-3.0 + 2.0 * torch.rand(U, generator=gen, device="cuda:0")) / c
    K[:, 1024, 0] = 0.0
    K[:, 1088, 0] = -int(24.0 / c)
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 1.0, 0.5, forced_policy=3))
    fg.fastgen_profile(Q, K, cls)
    fg.fastgen_compact(K, K)
    got = fg.fastgen_export_state()["scores"][:U * n].view(U, n)[:, 1024].cpu()
    fg.close()
    weight = torch.exp2(K[:, :, 0].double().cpu() * c)
    start = weight[:, 0] + weight[:, 1024]
    want = 64.0 / start + 192.0 / (start + weight[:, 1088])
    error = float(((got - want) / want).mean())
    print(f"row sums behind the one pass, U={U} d={d}: {error:.2e}")
    assert abs(error) < 1e-8


# A head none of whose rows fit the shifts of the rows 64 before costs no more than the maxima of its rows: each block is
# contracted once. Going through every block twice took 1.5 times an ordinary head's time at d = 128 and 1.6 at 64, so 1.15.
@pytest.mark.parametrize("U,n,d", [(700, 1000, 64), (1024, 1000, 128)])
def test_one_pass_of_rows_that_never_fit_costs_their_maxima(U, n, d):
    gen = torch.Generator(device="cuda:0").manual_seed(n + d)
    Q, K = (torch.randn(U, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
    cls = torch.ones((1, n), dtype=torch.uint8, device="cuda:0")
    cfg = binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 0.3, 0.3)
    space = torch.empty(binding.fastgen_workspace_bytes(cfg), dtype=torch.uint8, device="cuda:0")
    K[:, :, 0] = 8.0
    apart = torch.where((torch.arange(n, device="cuda:0") // 40) % 2 == 0, 32.0, -32.0).bfloat16()
    times = {0: [], 1: []}
    for _ in range(12):
        for jump in (0, 1):   # in turn: the clock is shared
            Q[:, :, 0] = apart * jump
            fg = binding.FastGen(cfg, "cuda:0", workspace=space)
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            fg.fastgen_profile(Q, K, cls)
            end.record()
            end.synchronize()
            times[jump].append(start.elapsed_time(end))
            fg.close()
    ratio = sorted(times[1])[4] / sorted(times[0])[4]
    print(f"rows that never fit, U={U} n={n} d={d}: {ratio:.2f}")
    assert ratio < 1.35


# Few heads with favoured columns (about 2^13 over the others, one in 16) are contracted once as heads without any are: a block
# done again costs 2 us of a call of 15 to 22 (1.08 to 1.14 times; without, 0.98 to 1.00).
@pytest.mark.parametrize("U,n,d", [(50, 435, 128), (64, 700, 128), (100, 200, 128)])
def test_one_pass_of_favoured_columns_costs_as_others(U, n, d):
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    plain = [torch.randn(U, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(2)]
    favoured = [x.clone() for x in plain]
    size = math.sqrt(9.0 * math.sqrt(d))
    favoured[0][:, :, 0] = size
    favoured[1][:, :, 0] = size * (torch.arange(n, device="cuda:0") % 16 == 5)
    cls = torch.ones((1, n), dtype=torch.uint8, device="cuda:0")
    cfg = binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 0.3, 0.3)
    policy, kept = (torch.empty((U, k), dtype=torch.int32, device="cuda:0") for k in (1, 5))
    recovery = torch.empty((U, 5), dtype=torch.float64, device="cuda:0")
    times = {0: [], 1: []}
    for _ in range(8):
        for which, (Q, K) in enumerate((plain, favoured)):   # in turn: the clock is shared
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            start.record()
            for _ in range(200):
                binding.fastgen_profile_static(cfg, Q, K, cls, policy, recovery, kept)
            end.record()
            end.synchronize()
            times[which].append(start.elapsed_time(end))
    ratio = min(times[1]) / min(times[0])
    print(f"favoured columns, U={U} n={n} d={d}: {ratio:.3f}")
    assert ratio < 1.06


# grouped heads, per-unit step (vector ALU for two heads and float32, matrix cores for three to eight bf16 heads) and
# split-KV for more heads, probed steps included
@pytest.mark.parametrize("heads,n,S,d,dtype,G", [
    (3, 1, 3, 128, "bf16", 2), (3, 17, 5, 128, "bf16", 3), (3, 130, 9, 128, "bf16", 4), (3, 130, 9, 64, "bf16", 4),
    (3, 250, 6, 128, "bf16", 5), (3, 250, 6, 128, "bf16", 8), (2, 251, 6, 64, "bf16", 8), (3, 100, 6, 128, "f32", 2),
    (3, 100, 6, 64, "f32", 4), (3, 65, 6, 128, "f32", 7), (2, 100, 6, 128, "bf16", 9), (2, 508, 4, 128, "bf16", 4),
    (2, 509, 4, 128, "bf16", 4), (256, 520, 3, 64, "bf16", 4), (260, 40, 12, 128, "bf16", 2),
])
def test_grouped_decode_step_forms(heads, n, S, d, dtype, G):
    w = W["llama7b_b1"].scaled(name="grouped_forms", layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=d,
                               dtype=dtype, seed=400 + n)
    run = H.GpuRun(w, range(w.num_units), group_size=G)
    check = sorted({0, 1, 2, heads // 2, heads - 1} & set(range(heads)))
    rep = H.compare(run, check_units=check, probe_steps=(1,), cover_policies=1)
    H.log_report(f"grouped forms U={heads} n={n} S={S} d={d} {dtype} G={G}", rep)


# The split form of three to eight bf16 heads: a few long units, full caches earlier, and more than 4608 tokens
@pytest.mark.parametrize("heads,n,S,d,G,forced", [(3, 2300, 4, 128, 3, -1), (2, 1900, 4, 128, 5, 3), (2, 1300, 4, 128, 3, 4), (3, 1500, 3, 128, 4, 4),
                                                  (2, 2600, 4, 128, 6, -1), (2, 4650, 4, 64, 8, -1), (2, 4650, 3, 64, 7, 2)])
def test_split_grouped_steps(heads, n, S, d, G, forced):
    w = W["llama7b_b1"].scaled(name="grouped_split", layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=d,
                               dtype="bf16", seed=500 + n)
    run = H.GpuRun(w, range(w.num_units), group_size=G, forced_policy=forced)
    run.fg.fastgen_enable_timing(1)
    rep = H.compare(run, probe_steps=(1,))
    assert run.fg.fastgen_read_timing()["decode_update"][1] == S
    H.log_report(f"grouped split U={heads} n={n} S={S} d={d} G={G} forced={forced}", rep)


# float32 outputs of a grouped step: both forms of the step on the same inputs (which one runs depends
# on the tokens reserved), against softmax(q K^T) V in float64. The one-workgroup-per-unit form walks a
# whole unit with one accumulator per lane group, the split form 256 tokens at a time, so the first one
# must not be the worse: 1.1 covers the different order of the sums; one chain over all tokens of a
# lane group (n / 16 at d = 128) has 1.17 times the split form's error in the first case.
@pytest.mark.parametrize("U,n,d,G", [(24, 1000, 128, 2), (24, 500, 64, 4), (256, 2400, 128, 2)])
def test_grouped_float32_outputs_as_accurate_as_the_split_form(U, n, d, G):
    gen = torch.Generator(device="cuda:0").manual_seed(n + G)
    Q, K, V = (torch.randn(x, n, d, generator=gen, device="cuda:0") for x in (U * G, U, U))
    q, k, v = (torch.randn(x, d, generator=gen, device="cuda:0") for x in (U * G, U, U))
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    Kd, Vd = torch.cat([K, k[:, None]], 1).double(), torch.cat([V, v[:, None]], 1).double()
    s = (Kd[:, None] * q.view(U, G, 1, d).double()).sum(3) * float(torch.tensor(1.0 / math.sqrt(d), dtype=torch.float32))
    ref = (torch.softmax(s, 2)[..., None] * Vd[:, None]).sum(2).view(U * G, d)
    err = {}
    for form, S in (("unit", 1), ("split", 4700 - n)):
        fg = binding.FastGen(binding.make_config(U, 1, d, torch.float32, n, S, 0.95, 0.3, 0.3, forced_policy=4, group_size=G))
        fg.fastgen_profile(Q, K, cls)
        fg.fastgen_compact(K, V)
        out = fg.fastgen_decode_step(q, k, v, cls[:, 0])
        err[form] = float((out.double() - ref).norm() / ref.norm())
        fg.close()
    print(f"[accuracy] grouped float32 U={U} n={n} d={d} G={G}: {err}", flush=True)
    assert err["unit"] <= 1.1 * err["split"], err


# A step that finds no free slot in a unit's reservation leaves the cache alone and reports it. The
# reservations rule this out, so the test takes a unit's last free slots away in its step record
# (unit, 0, slots reserved, tokens held, offset, policy word, 0) inside the workspace.
@pytest.mark.parametrize("G", [1, 2])
def test_step_without_a_free_slot_is_reported(G):
    U, n, d = 3, 20, 64
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    Q, K = (torch.randn(x, n, d, generator=gen, device="cuda:0") for x in (U * G, U))
    q, k = (torch.randn(x, d, generator=gen, device="cuda:0") for x in (U * G, U))
    cls = torch.zeros((1, n), dtype=torch.uint8, device="cuda:0")
    fg = binding.FastGen(binding.make_config(U, 1, d, torch.float32, n, 4, 0.95, 0.3, 0.3, forced_policy=4, group_size=G))
    fg.workspace.zero_()
    fg.fastgen_profile(Q, K, cls)
    fg.fastgen_compact(K, K)
    words = fg.workspace[:fg.workspace.numel() // 32 * 32].view(torch.int32).view(-1, 8)
    record = (words[:, 0] < U) & (words[:, 1] == 0) & (words[:, 2] == n + 4) & (words[:, 3] == n) & (words[:, 5] == 0)
    rows = torch.nonzero(record).flatten()
    assert rows.numel() == U and sorted(words[rows, 0].tolist()) == list(range(U)), rows
    row = rows[words[rows, 0] == 1]
    words[row, 2] = n
    fg.fastgen_decode_step(q, k, k, cls[:, 0])
    st = fg.fastgen_export_state(lengths_only=True)
    assert int(st["status"].item()) == binding.FG_ECAP
    lengths = st["lengths"].tolist()   # the other units' workgroups may have seen the report and stopped
    assert lengths[1] == n and set(lengths) <= {n, n + 1}


# A local window over the whole prompt keeps every column in every row, as special tokens everywhere do:
# the band sums are then the column sums, term by term, and the two recoveries the same number. The one
# pass by one and by several workgroups per unit; in two sweeps the split stream with 32 and 64 owners, and 256-owner
# blocks singly (d = 64) and in pairs.
@pytest.mark.parametrize("U,n,d,G,sweeps", [
    (2, 33, 64, 1, 1), (32, 333, 128, 1, 1), (4, 300, 64, 4, 2), (3, 300, 128, 2, 1), (300, 400, 128, 1, 1), (2, 1033, 64, 1, 2),
    (16, 1100, 128, 1, 2), (9, 2049, 64, 1, 2), (4, 1100, 64, 4, 2), (100, 1032, 64, 1, 2), (100, 1032, 128, 1, 2), (200, 1100, 128, 1, 2)])
def test_band_over_the_whole_prompt_is_the_column_sum(U, n, d, G, sweeps):
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    Q, K = (torch.randn(x, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for x in (U * G, U))
    cls = torch.ones((1, n), dtype=torch.uint8, device="cuda:0")
    cfg = binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 1.0, 0.3, family=(8, 1, 0, 0), group_size=G)
    fg = binding.FastGen(cfg)
    fg.fastgen_enable_timing(1)
    _, recovery, _ = fg.fastgen_profile(Q, K, cls)
    rec = recovery.cpu()
    assert fg.fastgen_read_timing()["sweep2"][1] == sweeps - 1
    fg.close()
    assert torch.equal(rec[:, 0], rec[:, 1]), (rec[:, 0] - rec[:, 1]).abs().max()
    assert float((rec[:, 0] - 1.0).abs().max()) < 1e-6


# Rows of the attention map sum to 1. A float32 1/l per row is off by up to half an ulp, 1.7e-8 rms in
# either direction: over 10^4 rows and more the mean mass is within 4 x 1.7e-8 / 100 of 1 unless merging
# the waves of the split-stream sweep adds an error of one sign (one hardware exponential per merge: 1.7e-9).
@pytest.mark.parametrize("U,n,d", [(16, 1100, 128), (16, 1100, 64), (4, 1500, 64)])   # 64, 64 and 32 owners
def test_split_stream_row_masses_have_no_bias(U, n, d):
    masses = []
    for seed in range(8):
        gen = torch.Generator(device="cuda:0").manual_seed(seed)
        Q, K = (torch.randn(U, n, d, generator=gen, device="cuda:0", dtype=torch.bfloat16) for _ in range(2))
        cls = torch.ones((1, n), dtype=torch.uint8, device="cuda:0")
        fg = binding.FastGen(binding.make_config(U, 1, d, torch.bfloat16, n, 0, 0.95, 0.3, 0.3))
        fg.fastgen_enable_timing(1)
        _, recovery, _ = fg.fastgen_profile(Q, K, cls)
        masses.append(float(recovery[:, 0].mean()) - 1.0)
        assert fg.fastgen_read_timing()["sweep2"][1] == 1
        fg.close()
    print(f"[accuracy] row masses U={U} n={n} d={d}: mean {sum(masses) / 8:.2e}", flush=True)
    assert abs(sum(masses) / 8) < 7e-10, masses


# the grouped split form's update kernel: 512 threads up to 512 units, above them 256 while a unit fits
# their registers (3072 tokens)
@pytest.mark.parametrize("heads,n,S,G", [(257, 60, 6, 9), (512, 60, 6, 9), (513, 60, 6, 9), (513, 300, 4, 12), (513, 3068, 4, 9),
                                         (513, 3069, 4, 9)])
def test_grouped_update_kernel_sizes(heads, n, S, G):
    w = W["llama7b_b1"].scaled(name="grouped_update", layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=64,
                               dtype="bf16", seed=300 + n)
    run = H.GpuRun(w, range(w.num_units), group_size=G, forced_policy=2)
    rep = H.compare(run, check_units=[0, heads - 1], probe_steps=(1,))
    H.log_report(f"grouped update U={heads} n={n} S={S} G={G}", rep)


# selection of many units: ten slots of 256 threads up to 2560 tokens, twelve of 512 up to 6144
@pytest.mark.parametrize("heads,n", [(513, 2560), (513, 2561), (513, 4097), (513, 6144), (513, 6145)])
def test_selection_sizes_of_many_units(heads, n):
    w = W["llama7b_b1"].scaled(name="selection_many", layers=1, heads=heads, batch=1, prompt_len=n, steps=1, head_dim=64,
                               seed=200 + n)
    run = H.GpuRun(w, range(w.num_units))
    rep = H.compare(run, check_units=[0, heads - 1])
    H.log_report(f"selection U={heads} n={n}", rep)


# decode units ordered by size up to 1024 of them, up to 4096 with 512 tokens or more, up to 16384 with 256 KiB
# or more (1024 tokens at d = 64)
@pytest.mark.parametrize("heads,n,S", [(1025, 508, 3), (1025, 509, 3), (4096, 509, 3), (4097, 509, 3), (4097, 1020, 3), (4097, 1021, 3)])
def test_order_of_decode_units(heads, n, S):
    w = W["llama7b_b1"].scaled(name="unit_order", layers=1, heads=heads, batch=1, prompt_len=n, steps=S, head_dim=64,
                               seed=100 + n)
    run = H.GpuRun(w, range(w.num_units))
    rep = H.compare(run, check_units=[0, 1, heads // 2, heads - 1], cover_policies=1)
    H.log_report(f"unit order U={heads} n={n} S={S}", rep)


# The update inside the one-workgroup-per-unit step holds 1, 2, 4, 8 or 12 tokens per thread: scored units on
# both sides of 512, 1024, 2048 and 4096 held tokens, plain and with grouped heads (256 units and more, so
# that the length does not send them to the split form), bf16 and float32. r = 1 keeps every token of a
# frequent + local policy, which still keeps scores; under r = 0.97 tokens leave.
@pytest.mark.parametrize("heads,n,d,dtype,G", [
    (256, 510, 64, "bf16", 2), (256, 1022, 64, "bf16", 2), (256, 2046, 64, "bf16", 2), (256, 2046, 64, "f32", 2),
    (256, 4094, 64, "bf16", 4), (256, 4500, 64, "bf16", 2), (256, 2040, 64, "bf16", 8), (256, 1022, 128, "f32", 4),
    (256, 2046, 64, "bf16", 1), (256, 4094, 64, "bf16", 1), (256, 4600, 64, "bf16", 1), (256, 4094, 64, "f32", 1),
])
@pytest.mark.parametrize("ratio", [1.0, 0.97])
def test_update_slots_of_long_scored_units(heads, n, d, dtype, G, ratio):
    w = W["llama7b_b1"].scaled(name="update_slots", layers=1, heads=heads, batch=1, prompt_len=n, steps=4, head_dim=d,
                               dtype=dtype, seed=n + G, r_l=ratio if ratio < 1 else 0.5, r_f=ratio)
    run = H.GpuRun(w, range(w.num_units), group_size=G, forced_policy=3)
    rep = H.compare(run, check_units=[0, heads - 1], probe_steps=(3,))
    lengths = run.fg.fastgen_export_state(lengths_only=True)["lengths"]
    assert int(lengths.min()) >= 0.97 * n
    assert ratio < 1 or int(lengths.min()) == n + 4
    H.log_report(f"update slots U={heads} n={n} d={d} {dtype} G={G} r={ratio}", rep)


# read-back by several workgroups per unit (few units) and by one (2048 units and more), rows included
@pytest.mark.parametrize("heads,n", [(1, 511), (1, 512), (3, 5000), (7, 2049), (2047, 300), (2048, 600)])
def test_read_back_by_several_workgroups(heads, n):
    w = W["llama7b_b1"].scaled(name="read_back", layers=1, heads=heads, batch=1, prompt_len=n, steps=2, head_dim=64,
                               seed=50 + n)
    run = H.GpuRun(w, range(w.num_units))
    run.profile_and_compact()
    states, off, keys, values = run.state(rows=True)
    lengths = run.fg.fastgen_export_state(lengths_only=True)["lengths"].tolist()
    pos = torch.cat([torch.from_numpy(p) for p, _ in states]).long().to(keys.device)
    unit = torch.repeat_interleave(torch.arange(heads), torch.tensor(lengths)).to(keys.device)
    assert off[-1] == sum(lengths) == pos.numel()
    assert bool(((pos[1:] > pos[:-1]) | (unit[1:] != unit[:-1])).all())
    assert torch.equal(keys, run.K[unit, pos]) and torch.equal(values, run.V[unit, pos])


# Nothing of what the workspace held before counts, rows behind the end of a unit or of a head in a partly filled
# tile included: a workspace of NaN patterns gives what a cleared one gives. The last six take the first 1024 columns in one
# pass, which leaves most statistics of the first 1024 rows unwritten, and the triangle behind them in the split stream with 32
# (two) and 64 owners, in blocks and in pairs (two).
@pytest.mark.parametrize("U,n,d,dtype,G", [(3, 5, 64, "bf16", 1), (3, 37, 128, "f32", 1), (2, 21, 64, "bf16", 3), (2, 1100, 128, "bf16", 2),
                                           (40, 333, 128, "bf16", 1), (2, 5000, 64, "bf16", 1),
                                           (16, 1100, 64, "bf16", 2), (13, 1500, 128, "bf16", 4), (64, 1313, 64, "bf16", 2),
                                           (300, 1313, 64, "bf16", 2), (200, 1999, 64, "bf16", 3), (128, 1999, 128, "bf16", 2)])
def test_previous_contents_of_the_workspace_are_not_read(U, n, d, dtype, G):
    w = W["llama7b_b1"].scaled(name="stale", layers=1, heads=U, batch=1, prompt_len=n, steps=3, head_dim=d, dtype=dtype, seed=n)
    seen = []
    for fill in (0, 255):
        run = H.GpuRun(w, range(U), group_size=G)
        run.fg.workspace.fill_(fill)
        pol, rec, cnt = run.profile_and_compact()
        outs = [run.step(t) for t in range(3)]
        st = run.fg.fastgen_export_state(rows=True)
        seen.append([torch.from_numpy(rec), torch.from_numpy(cnt)] + outs + [st[k] for k in ("positions", "scores", "keys", "values")])
        assert bool(torch.isfinite(torch.stack(outs).float()).all())
    assert all(torch.equal(a, b) for a, b in zip(*seen))
