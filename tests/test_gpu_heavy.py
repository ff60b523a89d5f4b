"""Unchecked graphs (validate = 0) whose node weights sum past 2^31 - 1, while every
label's weight stays within 32 bits: the candidates of one target can weigh more
than that.  Integer results, compared with the oracle element by element."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def sc():
    import paper_1404_4797_amd as m
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m.load()
    return m


def star(leaves):
    w = np.random.default_rng(1).integers(1, 500, size=leaves).astype(np.int32)
    return {"n": leaves + 1, "xadj": np.concatenate([[0], leaves + np.arange(leaves + 1)]).astype(np.int64),
            "adjncy": np.concatenate([np.arange(1, leaves + 1), np.zeros(leaves)]).astype(np.int32),
            "adjwgt": np.concatenate([w, w])}


# leaves: segments for one wave, for one workgroup and, with small select_small_max, for several; colours that count their
# candidates during evaluation and those that do not
GRAPHS = {"star_60": lambda: star(60), "star_3000": lambda: star(3000), "star_140001": lambda: star(140001),
          "ba": lambda: synth.ba(20000, 4, seed=3, weighted=True), "rmat": lambda: synth.rmat(14, 16, seed=3, weighted=True)}


def heavy(name):
    g = GRAPHS[name]()
    top = min((1 << 31) - 1, (1 << 36) // g["n"])
    g["vwgt"] = np.random.default_rng(2).integers(top // 2, top, size=g["n"]).astype(np.int32)
    assert g["vwgt"].astype(np.int64).sum() > 1 << 34
    return g


@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("knobs", [dict(), dict(select_small_max=1), dict(select_small_max=3, select_launches=1), dict(fused_eval=-1)])
def test_heavy_nodes(sc, name, knobs):
    g = heavy(name)
    d, n, cmax = sc.to_device(g), g["n"], int(g["vwgt"].max())
    for U in (cmax, min(5 * cmax, (1 << 31) - 1), (1 << 31) - 1):
        lab, rr = sc.cluster_dev(d, U, rounds=3, seed=5, validate=0, subrounds=2, **knobs)
        ref, rr_ref, _ = oracle.cluster(g, U, rounds=3, seed=5, nsub=2)
        assert rr == rr_ref and np.array_equal(lab.cpu().numpy(), ref), U
    for k in (64, 300, 2000):
        part = np.random.default_rng(k).integers(0, k, size=n).astype(np.int32)
        bw = np.bincount(part, weights=g["vwgt"], minlength=k)
        if bw.max() >= (1 << 31) / 1.1:
            continue
        for lmax in (int(bw.max() * 1.05), int(bw.mean() * 1.01) + cmax // 2):
            p, rr = sc.refine_dev(d, k, lmax, torch.from_numpy(part.copy()).cuda(), rounds=3, seed=5, validate=0,
                                  subrounds=2, **knobs)
            ref, rr_ref, _ = oracle.refine(g, k, lmax, part, rounds=3, seed=5, nsub=2)
            assert rr == rr_ref and np.array_equal(p.cpu().numpy(), ref), (k, lmax)


def test_an_unchecked_batch_may_weigh_more_than_one_graph(sc):
    gs = [{**synth.ba(3000, 4, seed=i, weighted=True), "vwgt": np.full(3000, 500_000, dtype=np.int32)} for i in range(4)]
    u, base = sc.union(gs)
    r = sc.partition_batch_dev(sc.to_device(u), base, [8] * 4, [0.05] * 4, [1, 2, 3, 4], validate=0, coarsest_nodes=500)
    for i, g in enumerate(gs):
        ref = oracle.partition(g, 8, 0.05, 1 + i, coarsest_nodes=500)
        assert np.array_equal(r["part"][base[i]:base[i + 1]].cpu().numpy(), ref["part"]) and r["cut"][i] == ref["cut"]
