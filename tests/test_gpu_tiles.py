"""Slot-parallel kernels (validation, cut, block weights, contraction) at the sizes where a
tile of 2048 slots, a thread's 8 slots or a workgroup's run of tiles ends, and
on arrays that do not start on a 16-byte boundary.  Compared with the oracle."""
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


def path_with_gaps(slots, seed):
    """A path of slots / 2 edges among nodes without neighbours, random weights."""
    edges = slots // 2
    rng = np.random.default_rng(seed)
    ids = np.sort(rng.choice(3 * edges + 5, size=edges + 1, replace=False))
    n = 3 * edges + 5
    w = rng.integers(1, 9, size=edges)
    src, dst = np.concatenate([ids[:-1], ids[1:]]), np.concatenate([ids[1:], ids[:-1]])
    wt = np.concatenate([w, w])
    order = np.argsort(src * n + dst)
    xadj = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int64)
    return {"n": n, "xadj": xadj, "adjncy": dst[order].astype(np.int32), "adjwgt": wt[order].astype(np.int32),
            "vwgt": rng.integers(0, 4, size=n).astype(np.int32)}


def shifted(t):
    """The same values from an address 4 bytes past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    buf[1:] = t
    return buf[1:]


GRAPHS = {**{"path_%d" % s: (lambda s=s: path_with_gaps(s, s)) for s in (2, 6, 8, 10, 2046, 2048, 2050, 4096, 6200)},
          "rmat_14": lambda: synth.rmat(14, 16, seed=5, weighted=True), "rgg": lambda: synth.rgg(40000, seed=6)}


@pytest.mark.parametrize("gname", list(GRAPHS))
@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("shift", [False, True])
def test_cut_and_validate(sc, gname, unit, shift):
    g = GRAPHS[gname]()
    if unit:
        g = {**g, "adjwgt": None, "vwgt": None}
    d = sc.to_device(g)
    if shift:
        for key in ("adjncy", "adjwgt", "vwgt"):
            d[key] = None if d[key] is None else shifted(d[key])
    assert sc.validate_dev(d) == 0
    for k in (2, 256, 257, 1024, 1025):
        part = np.random.default_rng(k).integers(0, k, size=g["n"]).astype(np.int32)
        dp = torch.from_numpy(part).cuda()
        cut, bw = sc.cut_dev(d, dp, k)
        ref_cut, ref_bw = oracle.cut(g, part, k)
        assert cut == ref_cut and np.array_equal(bw, ref_bw)
        assert (cut, list(bw)) == (lambda r: (r[0], list(r[1])))(sc.cut_dev_noalloc(d, dp, k))
        dp[g["n"] // 2] = k
        with pytest.raises(sc.SclapError):
            sc.cut_dev(d, dp, k)


@pytest.mark.parametrize("what", ["one weight", "one direction", "one id", "self-loop", "zero weight", "first offset"])
def test_broken_graphs(sc, what):
    g = GRAPHS["rmat_14"]()
    d = sc.to_device(g)
    e = len(g["adjncy"]) // 2 + 3
    row = int(np.searchsorted(g["xadj"], e, side="right")) - 1
    if what == "one weight":
        d["adjwgt"][e] += 1
        expect = sc.ERR_NOT_SYMMETRIC
    elif what == "one direction":  # (u, v) becomes (u, v') with v' on the same side of u and not equal to it
        v = int(g["adjncy"][e])
        d["adjncy"][e] = v - 1 if v - 1 > row or v < row and v > 0 else v + 1
        expect = sc.ERR_NOT_SYMMETRIC
    elif what == "one id":
        d["adjncy"][e] = g["n"]
        expect = sc.ERR_INVALID
    elif what == "self-loop":
        d["adjncy"][e] = row
        expect = sc.ERR_INVALID
    elif what == "zero weight":
        d["adjwgt"][e] = 0
        expect = sc.ERR_INVALID
    else:
        d["xadj"][0] = 1
        expect = sc.ERR_INVALID
    assert sc.validate_dev(d) == expect


def test_project_range(sc):
    C = torch.arange(5000, dtype=torch.int32, device="cuda") // 3
    coarse = torch.randint(0, 9, (1667,), dtype=torch.int32, device="cuda")
    assert torch.equal(sc.project_dev(C, coarse), coarse[C.long()])
    for bad in (-1, 1667):
        C[4321] = bad
        with pytest.raises(sc.SclapError):
            sc.project_dev(C, coarse)


def fans(lengths):
    """Node i joined to lengths[i] leaves of its own (one shared by all), rows of exactly those lengths first."""
    k = len(lengths)
    src = np.repeat(np.arange(k), lengths)
    dst = np.concatenate([np.r_[k, k + 1 + sum(lengths[:i]) + np.arange(d - 1)] for i, d in enumerate(lengths) if d])
    n = int(dst.max()) + 3
    u, v = np.concatenate([src, dst]), np.concatenate([dst, src])
    order = np.argsort(u * n + v)
    w = np.concatenate([1 + src % 7, 1 + src % 7])[order].astype(np.int32)
    xadj = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=n))]).astype(np.int64)
    return {"n": n, "xadj": xadj, "adjncy": v[order].astype(np.int32), "adjwgt": w, "vwgt": np.ones(n, dtype=np.int32)}


@pytest.mark.parametrize("lengths", [[1], [2047, 1, 2048], [2048, 2048, 1], [0, 2049, 0, 2047], [5000, 3, 1093, 2, 64],
                                     [6144, 0, 0, 1], [700, 1348, 1, 1, 9000]])
@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("group", [1, 2, 5])
def test_contract_tiles(sc, lengths, unit, group):
    g = fans(lengths)
    if unit:
        g = {**g, "adjwgt": None, "vwgt": None}
    labels = (np.arange(g["n"]) // group * group).astype(np.int32)
    C, cg = sc.contract_dev(sc.to_device(g), torch.from_numpy(labels).cuda())
    ref_C, ref = oracle.contract(g, labels)
    assert np.array_equal(C.cpu().numpy(), ref_C)
    for key in ("xadj", "adjncy", "adjwgt", "vwgt"):
        assert np.array_equal(cg[key].cpu().numpy(), ref[key]), key


@pytest.mark.parametrize("n", [1, 256, 257, 100003])
def test_refused_projection_writes_nothing(sc, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    coarse = torch.randint(0, 100, (50,), generator=gen, device="cuda", dtype=torch.int32)
    C = torch.randint(0, 50, (n,), generator=gen, device="cuda", dtype=torch.int32)
    expect = coarse[C.long()]
    for at, id_ in ((0, 50), (n // 2, -1), (n - 1, 1 << 30)):
        bad = C.clone()
        bad[at] = id_
        before, part = bad.clone(), torch.full((n,), 7, device="cuda", dtype=torch.int32)
        with pytest.raises(sc.SclapError):
            sc.project_dev(bad, coarse, part=part)
        assert bool((part == 7).all())
        with pytest.raises(sc.SclapError):
            sc.project_dev(bad, coarse, part=bad)
        assert torch.equal(bad, before)
    assert torch.equal(sc.project_dev(C, coarse, part=C), expect) and torch.equal(C, expect)
