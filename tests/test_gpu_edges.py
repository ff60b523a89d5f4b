"""Evaluation and admission at the sizes where their kernels change: row lengths
around every bucket, segment lengths around one
wave, one entry per thread, one workgroup's limit, and colours and label spaces
around the limits of the per-thread entry counts and of the direct LDS sums.
Integer results, compared with the oracle element by element."""
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


def star(leaves, seed):
    """Node 0 joined to every leaf: all leaves of a colour want the same label, so they form one segment."""
    rng = np.random.default_rng(seed)
    w = rng.integers(1, 5000, size=leaves).astype(np.int32)
    xadj = np.concatenate([[0], leaves + np.arange(leaves + 1)]).astype(np.int64)
    adj = np.concatenate([np.arange(1, leaves + 1), np.zeros(leaves)]).astype(np.int32)
    vw = rng.integers(0, 4, size=leaves + 1).astype(np.int32)
    return {"n": leaves + 1, "xadj": xadj, "adjncy": adj, "adjwgt": np.concatenate([w, w]), "vwgt": vw}


@pytest.mark.parametrize("leaves", [1, 2, 63, 64, 65, 256, 257, 512, 513, 1023, 1024, 1025, 16384, 16385, 65536, 65537, 70001, 262145])
@pytest.mark.parametrize("knobs", [dict(), dict(select_small_max=64), dict(select_small_max=1, select_launches=1)])
def test_one_segment(sc, leaves, knobs):
    g = star(leaves, leaves)
    color = np.zeros(leaves + 1, dtype=np.int32)
    color[0] = 1
    U = max(int(g["vwgt"].max()), int(g["vwgt"].sum()) // 2)
    lab, rr = sc.cluster_dev(sc.to_device(g), U, rounds=2, seed=3, color_override=torch.from_numpy(color).cuda(),
                             subrounds=2, **knobs)
    ref, rr_ref, _ = oracle.cluster(g, U, rounds=2, seed=3, nsub=2, color_override=color)
    assert rr == rr_ref and np.array_equal(lab.cpu().numpy(), ref)


@pytest.mark.parametrize("k", [2, 64, 257, 1024, 1025, 4096, 4097])
@pytest.mark.parametrize("n", [3000, 70000, 400000])
def test_label_spaces(sc, n, k):
    g = synth.ba(n, 4, seed=k, weighted=True)
    rng = np.random.default_rng(k)
    # uneven blocks, so that some cannot take what wants to join them
    part = np.minimum(rng.integers(0, k, size=n), rng.integers(0, k, size=n)).astype(np.int32)
    lmax = int(np.bincount(part, minlength=k).max())
    p, rr = sc.refine_dev(sc.to_device(g), k, lmax, torch.from_numpy(part.copy()).cuda(), rounds=2, seed=k, subrounds=1)
    ref, rr_ref, _ = oracle.refine(g, k, lmax, part, rounds=2, seed=k, nsub=1)
    assert rr == rr_ref and np.array_equal(p.cpu().numpy(), ref)


def centres(n, degrees, seed):
    """One node per entry of ``degrees`` joined to that many others, every bucket's first and last row length."""
    rng = np.random.default_rng(seed)
    k = len(degrees)
    u = np.repeat(np.arange(k), degrees)
    v = np.concatenate([k + rng.choice(n - k, size=d, replace=False) for d in degrees])
    w = rng.integers(1, 5, size=len(u))
    src, dst, wt = np.concatenate([u, v]), np.concatenate([v, u]), np.concatenate([w, w])
    order = np.argsort(src * n + dst)
    xadj = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int64)
    return {"n": n, "xadj": xadj, "adjncy": dst[order].astype(np.int32), "adjwgt": wt[order].astype(np.int32),
            "vwgt": np.ones(n, dtype=np.int32)}


DEGREES = [1, 4, 5, 16, 17, 32, 33, 64, 65, 256, 257, 1024, 1025, 4096, 4097, 8192, 8193, 16385, 25000]


@pytest.mark.parametrize("k", [0, 1, 3, 8, 16, 64, 65, 300])
@pytest.mark.parametrize("knobs", [dict(), dict(lane_max_degree=16), dict(fused_eval=-1), dict(block_table=16384),
                                   dict(hub_part_limit=1), dict(skip_quiet=1)])
def test_row_lengths(sc, k, knobs):
    g = centres(30000, DEGREES, 7)
    d = sc.to_device(g)
    for nsub in (1, 4):
        if k == 0:  # clustering
            lab, rr = sc.cluster_dev(d, 40, rounds=3, seed=5, subrounds=nsub, **knobs)
            ref, rr_ref, _ = oracle.cluster(g, 40, rounds=3, seed=5, nsub=nsub)
        else:
            part = np.random.default_rng(k).integers(0, k, size=g["n"]).astype(np.int32)
            lmax = -(-g["n"] // k) + g["n"] // (8 * k)
            lab, rr = sc.refine_dev(d, k, lmax, torch.from_numpy(part.copy()).cuda(), rounds=3, seed=5, subrounds=nsub,
                                    **knobs)
            ref, rr_ref, _ = oracle.refine(g, k, lmax, part, rounds=3, seed=5, nsub=nsub)
        assert rr == rr_ref and np.array_equal(lab.cpu().numpy(), ref)


def test_contracted_row_lengths(sc):
    # singleton clusters: every row passes the merge and the ordering and comes out as it went in
    g = centres(60000, [1, 2, 63, 64, 65, 256, 257, 512, 513, 2047, 2048, 2049, 4096, 4097, 8191, 8192, 8193, 16385, 50000],
                11)
    d = sc.to_device(g)
    C, cg = sc.contract_dev(d, torch.arange(g["n"], dtype=torch.int32, device="cuda"))
    assert torch.equal(C.cpu(), torch.arange(g["n"], dtype=torch.int32))
    for key in ("xadj", "adjncy", "adjwgt", "vwgt"):
        assert np.array_equal(cg[key].cpu().numpy(), g[key]), key
    # pairs of nodes: parallel edges merge
    lab = torch.arange(g["n"], dtype=torch.int32, device="cuda") // 2
    C, cg = sc.contract_dev(d, lab)
    ref_C, ref = oracle.contract(g, lab.cpu().numpy())
    assert np.array_equal(C.cpu().numpy(), ref_C)
    for key in ("xadj", "adjncy", "adjwgt", "vwgt"):
        assert np.array_equal(cg[key].cpu().numpy(), ref[key]), key
