"""The sizes at which a kernel's work changes hands: cache lengths around the
32-row tiles and the four-wave parts of the one-launch context pass, and rows of
visual tokens around the key counts that a selecting thread holds in registers
(2, 4, ..., 32 keys of 1024 threads; more stay in LDS or memory).

Tolerances: real outputs against the fp64 reference as in _parity; the masses of
the call without V against those with V to 4e-6 (a few fp32 ulps: separately
compiled kernels); selections are exact."""
import numpy as np
import pytest
import torch

from _parity import assert_step_equals_calls, check_sequence, kept_in_merge, own_text_parts, small_workload, tile_batch
from oracle import plant as P
from oracle import vp_oracle as O
from paper_2605_31457_amd import step as S

pytestmark = pytest.mark.gpu


def _check(tag, w, ref, n_ref, max_vis=None):
    ds = S.DeviceStep(w) if max_vis is None else S.DeviceStep(w, max_vis=max_vis)
    ds.decode_step()
    g = ds.results()
    ds.run(fused=True)
    assert_step_equals_calls(g, ds.results(), True, kept_in_merge(ds), tag)
    for b in range(w.B):
        check_sequence(tag, w, g, b, ref[b % n_ref], b_src=b % n_ref)
    return ds, g


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 28, 4, 128), ("bf16", 4, 1, 64), ("f32", 4, 2, 128), ("f32", 4, 1, 64)])
def test_lengths_around_tiles_and_parts(dtype, Hq, Hkv, d):
    """Waves of a part with no tile, one tile or an odd visual tile left over;
    segments that begin and end on, before and after a tile's edge."""
    lens = [1, 31, 32, 33, 64, 95, 128, 129, 160, 257, 1023, 1057]
    segs = [[(0, 1)], [], [(0, 32)], [(31, 2)], [(0, 32)], [(1, 63)], [(32, 64)], [(0, 97)], [(31, 1), (33, 63)],
            [(0, 256)], [(14, 500), (514, 31), (546, 400)], [(33, 1023)]]
    w = small_workload(seed=71, B=len(lens), Hq=Hq, Hkv=Hkv, d=d, lens=lens, segs=segs, dtype=dtype, S_cap=1100)
    ref, _ = P.plant(w, P.params_of(w))
    ds, g = _check(f"edges {dtype} d={d}", w, ref, w.B)
    ds.run(fused=False)  # no V in the mass call: statistics alone in the one launch
    n = ds.results()
    for key in ("mass_head", "mass_seq", "scores"):
        np.testing.assert_allclose(n[key], g[key], rtol=4e-6, atol=1e-30, err_msg=key)
    for key in ("k", "vis_idx"):
        assert np.array_equal(n[key], g[key]), key


@pytest.mark.parametrize("B,Hkv,d", [(64, 4, 64), (65, 4, 128), (128, 4, 64), (513, 1, 64)])
def test_many_sequence_and_kv_head_pairs(B, Hkv, d):
    """256 pairs and fewer share a resident round of four-wave parts; more take two
    parts (one from 512 pairs), and single-wave ones in a later layer's text pass,
    whose own text rows the call without the workspace's text part reads."""
    base = small_workload(seed=76, B=3, Hq=4 * Hkv, Hkv=Hkv, d=d, lens=[290, 33, 150],
                          segs=[[(20, 100), (130, 31)], [(1, 31)], []])
    ref, _ = P.plant(base, P.params_of(base))
    w = tile_batch(base, B)
    ds, g = _check(f"{B} x {Hkv}", w, ref, 3)
    ds.run(fused=False)
    n = ds.results()
    assert own_text_parts(ds) or B * Hkv <= 256
    assert_step_equals_calls(g, n, False, kept_in_merge(ds) or own_text_parts(ds), f"{B} x {Hkv} own text")
    for b in range(w.B):
        check_sequence(f"{B} x {Hkv} own text", w, n, b, ref[b % 3], b_src=b % 3)


@pytest.mark.parametrize("n_vis", [2047, 2048, 2049, 4097, 8192, 8193, 16385, 32768, 32769])
def test_step_selection_around_the_keys_a_thread_holds(n_vis):
    w = small_workload(seed=72, B=2, Hq=4, Hkv=1, d=64, lens=[n_vis + 60, 200], segs=[[(30, n_vis)], [(20, 150)]])
    ref, _ = P.plant(w, P.params_of(w))
    _check(f"{n_vis} visual tokens", w, ref, w.B)


@pytest.mark.parametrize("n_vis", [1000, 2049, 9000, 20000])
def test_step_selection_with_one_work_group_per_row(n_vis):
    """256 rows: each row's keys go from LDS to registers in one work-group."""
    base = small_workload(seed=73, B=2, Hq=4, Hkv=1, d=64, lens=[n_vis + 60, 200], segs=[[(30, n_vis)], [(20, 150)]])
    ref, _ = P.plant(base, P.params_of(base))
    _check(f"256 rows of {n_vis}", tile_batch(base, 256), ref, 2, max_vis=n_vis)


def test_step_selection_with_one_work_group_per_row_past_the_lds():
    """256 rows with room for 32000 keys each, more than a work-group's LDS but not than
    its registers hold: the row's keys take the general path, in LDS where they fit."""
    base = small_workload(seed=80, B=2, Hq=4, Hkv=1, d=64, lens=[3000, 200], segs=[[(30, 2900)], [(20, 150)]])
    ref, _ = P.plant(base, P.params_of(base))
    _check("256 rows of 32000", tile_batch(base, 256), ref, 2, max_vis=32000)


@pytest.mark.parametrize("n", [1, 63, 2047, 2048, 2049, 4096, 4097, 8193, 16384, 16385, 32768, 32769])
def test_topk_around_the_keys_a_thread_holds(n):
    """Distinct, tied, equal and special scores; k from 0 over the count that fits
    the staged ranks to every token. The second row is shorter than the first."""
    rng = np.random.default_rng(74)
    n1 = max(1, n - 65)
    segs = [[(5, n)], [(5, n1)]]
    lens = [n + 10, n1 + 10]
    w = small_workload(seed=75, B=2, Hq=1, Hkv=1, d=64, lens=lens, segs=segs, spike=0)
    ds = S.DeviceStep(w, k_cap=n, max_vis=n)
    vis = [O.visual_positions(lens[b], segs[b]) for b in range(2)]
    for kind in ("distinct", "tied", "equal", "extreme"):
        sc = rng.random((2, n)).astype(np.float32)
        if kind == "tied":
            sc = (np.floor(sc * 16) / 16).astype(np.float32)
        elif kind == "equal":
            sc[:] = np.float32(1.0 / 7.0)
        elif kind == "extreme":  # zeros, the least and largest floats and +inf among the scores
            sc[:, ::3] = 0.0
            sc[:, 1::7] = np.float32(np.finfo(np.float32).tiny)
            sc[:, 2::11] = np.float32(np.finfo(np.float32).max)
            sc[:, 4::301] = np.inf
        for k in sorted({0, 1, n // 20, n // 2, n - 1, n}):
            ds.scores.copy_(torch.from_numpy(sc))
            ds.k.copy_(torch.tensor([k, k], dtype=torch.int32))
            ds.select_topk()
            got = ds.vis_idx.cpu().numpy()
            for b, nb in enumerate((n, n1)):
                kb = min(k, nb)
                want = O.select_top_k(sc[b, :nb].astype(np.float64), vis[b], kb)
                assert np.array_equal(got[b, :kb], want), (kind, k, b)
                assert np.all(got[b, kb:] == -1), (kind, k, b)


def _step_calls_and_own_text(tag, w, ref, n_ref):
    """The step against the reference and the calls, and the layer that reads its own
    text rows: the step's bits, except where the header says to rounding only."""
    ds, g = _check(tag, w, ref, n_ref)
    ds.run(fused=False)
    n = ds.results()
    assert own_text_parts(ds) or w.B * w.Hkv <= 256
    assert_step_equals_calls(g, n, False, kept_in_merge(ds) or own_text_parts(ds), tag)
    for b in range(w.B):
        check_sequence(f"{tag}, own text", w, n, b, ref[b % n_ref], b_src=b % n_ref)


@pytest.mark.parametrize("dtype,Hkv,d,B,L", [
    # fp32 rows of 128 (one four-wave work-group per CU): parts of one round, fewer
    # where the kept work-groups need slots, of two rounds with more pairs, one per
    # pair, two past a round, one again
    ("f32", 2, 128, 2, 2900), ("f32", 4, 128, 4, 3300), ("f32", 8, 128, 6, 745), ("f32", 4, 128, 9, 3600),
    ("f32", 4, 128, 40, 290), ("f32", 4, 128, 40, 800),
    ("f32", 4, 128, 64, 290), ("f32", 4, 128, 65, 290), ("f32", 4, 128, 96, 290), ("f32", 4, 128, 97, 290),
    # bf16: two parts above half a round, one from three quarters, two from seven
    # eighths, one at a round, two up to one and a half, one beyond
    ("bf16", 4, 64, 95, 290), ("bf16", 4, 64, 96, 290), ("bf16", 4, 64, 111, 290), ("bf16", 4, 64, 112, 290),
    ("bf16", 4, 64, 128, 290), ("bf16", 4, 64, 129, 290), ("bf16", 4, 64, 192, 290), ("bf16", 4, 64, 193, 290)])
def test_parts_per_pair(dtype, Hkv, d, B, L):
    base = small_workload(seed=77, B=3, Hq=2 * Hkv, Hkv=Hkv, d=d, lens=[L, 33, 150], dtype=dtype,
                          segs=[[(20, L // 3), (L // 2, L // 9)], [(1, 31)], []])
    ref, _ = P.plant(base, P.params_of(base))
    _step_calls_and_own_text(f"{dtype} {B} x {Hkv} x {L}", tile_batch(base, B), ref, 3)


@pytest.mark.parametrize("dtype,Hq,B,T", [("bf16", 8, 1, 1), ("bf16", 8, 10, 1), ("bf16", 8, 11, 1), ("bf16", 14, 7, 2),
                                          ("bf16", 14, 8, 2), ("f32", 4, 5, 1), ("f32", 4, 6, 1)])
def test_later_layer_work_group_order(dtype, Hq, B, T):
    """Text and kept work-groups in one launch: interleaved while the kept ones (here
    two per pair and query, rounded up) are at most a twelfth of a round, all of the
    text ones first beyond."""
    base = small_workload(seed=78, B=3, Hq=Hq, Hkv=2, d=128, lens=[1300, 700, 40], dtype=dtype,
                          segs=[[(20, 900), (1000, 37)], [(33, 500)], [(2, 30)]])
    ref, _ = P.plant(base, P.params_of(base))
    w = tile_batch(base, B)
    if T > 1:  # the other query: the heads in another order
        w.q = np.stack([w.q, np.roll(w.q, 1, axis=1)], axis=1)
    ds = S.DeviceStep(w, k_cap=170)
    ds.decode_step()
    g = ds.results()
    ds.run(fused=False)
    n = ds.results()
    assert not own_text_parts(ds)
    assert_step_equals_calls(g, n, False, kept_in_merge(ds), f"{dtype} {B} x 2, {T} queries")
    if T == 1:
        for b in range(B):
            check_sequence(f"{dtype} {B} x 2", w, n, b, ref[b % 3], b_src=b % 3)


@pytest.mark.parametrize("Hq,Hkv,d,B,L", [(4, 1, 64, 1, 33), (4, 1, 64, 1, 2048), (4, 1, 64, 1, 2049), (4, 1, 64, 16, 512),
                                          (4, 1, 64, 17, 512), (28, 4, 128, 1, 2048), (28, 4, 128, 2, 1025),
                                          (32, 8, 128, 2, 500)])
@pytest.mark.parametrize("block_size", [0, 16, 32])
def test_small_fp32_steps(Hq, Hkv, d, B, L, block_size):
    """fp32 steps of one tile per single-wave part (up to 64 tiles, 256 over the
    batch) and the four-wave parts next to them, contiguous and paged."""
    base = small_workload(seed=79, B=2, Hq=Hq, Hkv=Hkv, d=d, lens=[L, max(1, L // 2 - 5)], dtype="f32",
                          segs=[[(3, L // 2), (L // 2 + 7, L // 5)], [(0, L // 4)]])
    ref, _ = P.plant(base, P.params_of(base))
    w = tile_batch(base, B)
    ds = S.DeviceStep(w, block_size=block_size, block_seed=4)
    ds.decode_step()
    g = ds.results()
    for b in range(B):
        check_sequence(f"{B} x {Hkv} x {L}", w, g, b, ref[b % 2], b_src=b % 2)
    for fused in (True, False):
        ds.run(fused=fused)
        assert_step_equals_calls(g, ds.results(), fused, kept_in_merge(ds), f"{B} x {Hkv} x {L} fused={fused}")


@pytest.mark.parametrize("dtype,d,n_text,own", [("bf16", 128, 500, True), ("bf16", 128, 2040, True),
                                                ("bf16", 128, 2060, False), ("f32", 64, 2040, True),
                                                ("f32", 128, 1020, True), ("f32", 128, 1060, False)])
@pytest.mark.parametrize("block_size", [0, 16])
def test_later_layer_with_few_text_rows(dtype, d, n_text, own, block_size):
    """64 pairs whose four-wave parts fill a round: up to two tiles of text per wave the
    layer's own text rows go to single-wave parts, more to the step's parts."""
    base = small_workload(seed=82, B=2, Hq=16, Hkv=4, d=d, lens=[n_text + 900, 500], dtype=dtype,
                          segs=[[(40, 500), (600, 400)], [(3, 400)]])
    ref, _ = P.plant(base, P.params_of(base))
    w = tile_batch(base, 16)
    ds = S.DeviceStep(w, max_vis=900, block_size=block_size, block_seed=6)
    assert own_text_parts(ds) == own
    ds.decode_step()
    g = ds.results()
    ds.run(fused=False)
    n = ds.results()
    assert_step_equals_calls(g, n, False, kept_in_merge(ds) or own, f"{dtype} {n_text} text rows")
    for b in range(w.B):
        check_sequence(f"{dtype} {n_text} text rows", w, n, b, ref[b % 2], b_src=b % 2)
