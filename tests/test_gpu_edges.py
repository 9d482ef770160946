"""Shapes at the edges of the kernels' tiles and dispatch rules, against the float64 oracle."""
import pytest

import fg_harness as H
from paper_2310_01801_amd import synth

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
