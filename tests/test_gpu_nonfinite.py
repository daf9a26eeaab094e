"""Cache rows whose logits are -inf (a key row with an infinite component, as a program
writes it to switch a row off): they weigh nothing, whether they fill a wave's only
tile, its first tile, a lane's rows of a visual tile, or a single row. Against the fp64
reference, where exp(-inf) = 0."""
import numpy as np
import pytest

from _parity import check_sequence, small_workload, tile_batch
from oracle import plant as P
from paper_2605_31457_amd import step as S

pytestmark = pytest.mark.gpu


def _off(w, b, rows):
    """Every query of sequence b gets logit -inf for the given cache rows."""
    neg_inf = np.float32(-np.inf) if w.dtype == "f32" else np.uint16(0xFF80)
    if w.dtype == "f32":
        w.q[b, :, 0] = np.maximum(np.abs(w.q[b, :, 0]), np.float32(0.25))
    else:
        w.q[b, :, 0] = np.maximum(w.q[b, :, 0] & np.uint16(0x7FFF), np.uint16(0x3E80))  # |q|, at least 0.25
    w.K[b][:, rows, 0] = neg_inf


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 8, 2, 128), ("bf16", 4, 1, 64), ("f32", 4, 2, 128),
                                            ("f32", 4, 1, 64)])
@pytest.mark.parametrize("copies", [1, 64, 300])
def test_rows_with_logit_minus_inf(dtype, Hq, Hkv, d, copies):
    """One copy of the batch (a tile or two per wave), 64 and 300 of it (more (sequence,
    KV head) pairs, so a wave's first tile of -inf is followed by others)."""
    base = small_workload(seed=95, B=2, Hq=Hq, Hkv=Hkv, d=d, lens=[700, 330], dtype=dtype,
                          segs=[[(64, 300), (420, 90)], [(40, 200)]])
    _off(base, 0, np.r_[0:32, 64:128, 200, 512:544, 600])  # text tiles, visual tiles, single rows
    _off(base, 1, np.r_[0:40, 250:290, 329])
    with np.errstate(invalid="ignore"):
        ref, _ = P.plant(base, P.params_of(base))
    assert all(np.isfinite(r.out).all() and np.isfinite(r.mass_head).all() for r in ref.values())
    w = base if copies == 1 else tile_batch(base, 2 * copies)
    ds = S.DeviceStep(w)
    for tag, run in (("step", lambda: ds.decode_step()), ("own text", lambda: ds.run(fused=False))):
        run()
        g = ds.results()
        for b in range(w.B):
            check_sequence(f"{copies} copies, {tag}", w, g, b, ref[b % 2], b_src=b % 2)
