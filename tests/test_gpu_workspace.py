"""What a workspace held before a call does not reach its results: the calls run on
workspaces filled with 0xFF bytes (NaN as floats) and are compared with the fp64
reference, at shapes whose merge has more partials than a lane group holds in
registers (64 at head_dim 128, 128 at 64) and most of whose kept splits are empty."""
import numpy as np
import pytest

from _parity import check_sequence, small_workload
from oracle import plant as P
from paper_2605_31457_amd import step as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 4, 1, 128), ("f32", 4, 2, 128), ("bf16", 4, 1, 64),
                                            ("f32", 4, 1, 64)])
@pytest.mark.parametrize("long", [True, False])
def test_results_do_not_depend_on_the_workspace(dtype, Hq, Hkv, d, long):
    """Row capacities of 8192 kept tokens (256 splits of 32) for budgets of a few
    tokens, one of a few hundred, and none (a sequence without visual tokens); with
    `long`, a cache of enough parts to exceed the registers by itself."""
    lens = [17000 if long else 1500, 300, 90]
    segs = [[(20, 700)], [(10, 40), (100, 50)], []]
    w = small_workload(seed=91, B=3, Hq=Hq, Hkv=Hkv, d=d, lens=lens, segs=segs, dtype=dtype)
    ref, _ = P.plant(w, P.params_of(w))
    ds = S.DeviceStep(w, k_cap=8192)
    for tag, run in (("step", lambda: ds.decode_step()), ("calls", lambda: ds.run(fused=True)),
                     ("own text", lambda: ds.run(fused=False))):
        ds.ws.fill_(0xFF)
        run()
        g = ds.results()
        for b in range(w.B):
            check_sequence(f"{tag} on a workspace of 0xFF bytes", w, g, b, ref[b])
    # a later layer: the kept lists are given, the workspace holds nothing of this layer
    ds.ws.fill_(0xFF)
    ds.out.fill_(7.0)
    ds.sparse_decode_attn(fused=False)
    later = ds.results()
    assert np.array_equal(later["out"], g["out"])
