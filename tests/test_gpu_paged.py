"""Paged KV caches (block tables, as serving engines keep them) through the C ABI.

The caches are cut into blocks of P rows dealt to physical blocks in a seeded
random order. The kernels gather the same rows into the same tiles as on the
contiguous caches, so every output is bit-identical to the contiguous run; the
planted workloads are also checked against the fp64 reference.
"""
import numpy as np
import pytest

from _parity import check_sequence, small_workload
from oracle import plant as P
from oracle import vp_oracle as O
from paper_2605_31457_amd import step as S
from paper_2605_31457_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("mass_head", "mass_seq", "scores", "k", "vis_idx", "out")


def _log(msg):
    print(msg, flush=True)


def _same(a, b, tag):
    for key in KEYS:
        assert np.array_equal(a[key], b[key]), f"{tag}: {key} differs from the contiguous run"


@pytest.mark.parametrize("bs", [16, 32, 256])
def test_paged_decode_step_config2(bs):
    w = W.generate(2)
    ref, _ = P.plant(w, P.params_of(w))
    flat = S.DeviceStep(w)
    flat.decode_step()
    a = flat.results()
    _log(f"cfg2 paged P={bs}")
    paged = S.DeviceStep(w, block_size=bs, block_seed=bs)
    paged.decode_step()
    g = paged.results()
    _same(a, g, f"cfg2 P={bs}")
    check_sequence(f"cfg2 paged P={bs}", w, g, 0, ref[0])
    # the four calls on the paged caches, fused and unfused text paths
    for fused in (True, False):
        paged.run(fused=fused)
        flat.run(fused=fused)
        _same(flat.results(), paged.results(), f"cfg2 P={bs} calls fused={fused}")


def test_paged_decode_step_config3_ragged():
    """16 ragged sequences (5120..12288 tokens), blocks of 64 rows."""
    w = W.generate(3)
    ref, _ = P.plant(w, P.params_of(w))
    flat = S.DeviceStep(w)
    flat.decode_step()
    paged = S.DeviceStep(w, block_size=64, block_seed=3)
    paged.decode_step()
    g = paged.results()
    _same(flat.results(), g, "cfg3 P=64")
    for b in range(w.B):
        check_sequence("cfg3 paged", w, g, b, ref[b])


PAGED_SMALL = {
    "f32-d64": (dict(seed=9, dtype="f32", B=2, Hq=4, Hkv=1, d=64, lens=[200, 45], segs=[[(16, 150)], [(0, 40)]]), 8),
    "short-seqs": (dict(seed=8, B=3, Hq=4, Hkv=1, d=64, lens=[1, 5, 31], segs=[[], [(1, 3)], [(0, 31)]]), 4),
    "many-segments": (dict(seed=4, B=2, Hq=28, Hkv=4, d=128, lens=[500, 450],
                           segs=[[(3, 50), (60, 40), (101, 7), (200, 100), (320, 90)],
                                 [(10, 10), (20, 10), (30, 300)]]), 16),
    "capacity-gt-len": (dict(seed=10, B=2, Hq=8, Hkv=1, d=128, lens=[70, 130], segs=[[(2, 60)], [(64, 64)]],
                             S_cap=200), 128),
}


@pytest.mark.parametrize("name", sorted(PAGED_SMALL))
def test_paged_small_shapes(name):
    spec, bs = PAGED_SMALL[name]
    w = small_workload(**spec)
    ref, _ = P.plant(w, P.params_of(w))
    flat = S.DeviceStep(w)
    flat.decode_step()
    paged = S.DeviceStep(w, block_size=bs, block_seed=7)
    paged.decode_step()
    g = paged.results()
    _same(flat.results(), g, f"{name} P={bs}")
    for b in range(w.B):
        check_sequence(f"{name} paged", w, g, b, ref[b])


def test_paged_later_layer_dense_attention():
    """A later layer's attention over the anchor's kept set, reading its own text
    rows from paged caches (vp_sparse_decode_attn without the workspace text),
    against the reference over the same context."""
    w = W.generate(2)
    ref, _ = P.plant(w, P.params_of(w))
    anchor = S.DeviceStep(w)
    anchor.decode_step()
    g = anchor.results()
    sel = g["vis_idx"][0, :int(g["k"][0])]
    wl = W.generate(2, seed=23)
    dl = S.DeviceStep(wl, block_size=32, block_seed=11)
    dl.vis_idx.copy_(anchor.vis_idx)
    dl.k.copy_(anchor.k)
    dl.sparse_decode_attn(fused=False)
    got = dl.results()["out"][0]
    L = int(wl.seq_len[0])
    J = np.sort(np.concatenate([sel, O.text_positions(L, wl.segments[0])]))
    qf = O.as_f64(wl.q[0])
    G = wl.Hq // wl.Hkv
    sm = 1.0 / np.sqrt(wl.d)
    want = np.stack([O.pruned_attention(qf[h], wl.K[0, h // G], wl.V[0, h // G], J, sm) for h in range(wl.Hq)])
    np.testing.assert_allclose(got, want, atol=2e-2, rtol=1e-2)


def test_paged_two_launch_plan():
    """A batch past the one-launch limit of the context pass (16 sequences x 64
    KV heads x 35 tiles > 32768 tiles), so the visual and text passes run as two
    launches, both reading rows through the block table: bit-identical to the
    contiguous caches and checked against the reference."""
    rng = np.random.default_rng(71)
    lens = [int(x) for x in rng.integers(1000, 1101, size=16)]
    segs = [[(10, 300), (400, 250)] for _ in range(16)]
    w = small_workload(seed=71, B=16, Hq=128, Hkv=64, d=64, lens=lens, segs=segs, S_cap=1100)
    ref, _ = P.plant(w, P.params_of(w))
    flat = S.DeviceStep(w)
    from paper_2605_31457_amd import vp
    assert not vp.vp_step_plan(flat.shape, flat.params) & vp.VP_PLAN_ONE_CONTEXT_LAUNCH
    flat.decode_step()
    a = flat.results()
    paged = S.DeviceStep(w, block_size=32, block_seed=5)
    paged.decode_step()
    g = paged.results()
    _same(a, g, "two-launch P=32")
    for b in range(w.B):
        check_sequence("paged two-launch", w, g, b, ref[b])
    for fused in (True, False):
        paged.run(fused=fused)
        flat.run(fused=fused)
        _same(flat.results(), paged.results(), f"two-launch P=32 calls fused={fused}")
    _log(f"paged two-launch: k={[ref[b].k for b in range(4)]}...")


EMPTY = {
    # kept rows in the merge launch; a kept pass (fp32); four-wave parts of several tiles
    "bf16-d128": (dict(seed=81, B=3, Hq=8, Hkv=2, d=128, lens=[70, 120, 90], segs=[[(5, 40)], [(10, 60)], [(0, 40)]]), 16),
    "f32-d64": (dict(seed=82, dtype="f32", B=3, Hq=4, Hkv=1, d=64, lens=[70, 120, 90],
                     segs=[[(5, 40)], [(10, 60)], [(0, 40)]]), 32),
    "f32-d128": (dict(seed=83, dtype="f32", B=3, Hq=4, Hkv=1, d=128, lens=[70, 400, 90],
                      segs=[[(5, 40)], [(10, 300)], [(0, 40)]]), 64),
    "bf16-d64-long": (dict(seed=84, B=3, Hq=16, Hkv=4, d=64, lens=[700, 1500, 900],
                           segs=[[(5, 400)], [(10, 1100)], [(0, 64), (100, 700)]]), 32),
}


@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("name", sorted(EMPTY))
def test_paged_zero_length_sequence(name, first):
    """A sequence of length 0 (the first of the batch, whose table row has nothing
    before it, or the last) uses no block, so its table entries name none (-1): the
    step, the four calls and a layer that reads its own text rows give the empty
    context's results for it and, for its neighbours, the bits of the contiguous
    caches."""
    spec, bs = EMPTY[name]
    w = small_workload(**spec)
    e = 0 if first else w.B - 1
    ref, _ = P.plant(w, P.params_of(w))
    flat = S.DeviceStep(w)
    paged = S.DeviceStep(w, block_size=bs, block_seed=9)
    for ds in (flat, paged):
        ds.seq_len[e] = 0
    paged.block_table[e] = -1
    for run in (lambda ds: ds.decode_step(), lambda ds: ds.run(fused=True), lambda ds: ds.run(fused=False)):
        got = []
        for ds in (flat, paged):
            ds.scores.fill_(-1.0)
            ds.out.fill_(7.0)
            run(ds)
            got.append(ds.results())
        _same(got[0], got[1], f"{name} with an empty sequence")
        g = got[1]
        for b in range(w.B):
            if b != e:
                check_sequence(f"{name} beside an empty sequence", w, g, b, ref[b])
        assert np.all(g["mass_head"][e] == 0.0) and np.all(g["mass_seq"][e] == 0.0)
        assert int(g["k"][e]) == 0 and np.all(g["vis_idx"][e] == -1)
        assert np.all(g["scores"][e] == -1.0), "no visual rank: no score is written"
        assert np.all(g["out"][e] == 0.0)
