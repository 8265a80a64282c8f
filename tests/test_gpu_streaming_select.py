"""The streaming select (queries grouped by direction, keys in superblocks with
bounds, loser trees) against the oracle, at sizes just past those that the dense
select takes.  Each test first asserts that its call goes to the streaming
kernel, so that a path line that moves fails here instead of emptying the test.
"""
import numpy as np
import pytest

import oracle
import workloads
from parity import allclose_report, check_sets_all, check_structure, sample_rows, stratified_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2604_03815_amd as kmip  # noqa: E402

DEV = torch.device("cuda:0")
FILL = 0x7F


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(DEV)


class PathProbe:
    """A filled workspace for one call on a single graph: the streaming kernel
    clears its counters, which lie behind the tiled keys (32 rows a tile, 16
    tiles more than the keys need); the dense select leaves them alone."""

    def __init__(self, N, H, d, k):
        self.ws = kmip.Workspace(DEV)
        self.ws.get(kmip.topk_workspace_size(N, H, d, k, 1)).fill_(FILL)
        self.at = (H * (-(-N // 32) + 16) * 32 * d * 2 + 255) // 256 * 256

    def streamed(self):
        counters = self.ws.buf[self.at:self.at + 512]
        return bool((counters != FILL).any())


@pytest.mark.parametrize("N,H,d,k,streams", [
    (300, 2, 16, 8, False), (9000, 2, 64, 128, False), (65536, 1, 16, 32, False), (65537, 1, 16, 32, True),
    (65536, 1, 128, 16, False), (65537, 1, 128, 16, True),
    # 32 < k < 64 at d = 128
    (32768, 2, 128, 33, False), (32769, 2, 128, 33, True), (32769, 2, 128, 64, False), (49152, 1, 128, 63, False), (49153, 1, 128, 63, True)])
def test_probe_tells_the_paths_apart(N, H, d, k, streams):
    p = PathProbe(N, H, d, k)
    q = torch.randn(N, H, d, device=DEV).bfloat16()
    kmip.topk(q, q, k, workspace=p.ws)
    torch.cuda.synchronize()
    assert p.streamed() == streams


def _far_clusters(N, H, d, k):
    # keys in 64 tight clusters far from the origin (|c| about 80, spread
    # 0.004): the rounding margin dominates a superblock's radius
    rng = np.random.default_rng(64)
    cen = rng.standard_normal((64, H, d)).astype(np.float32) * np.float32(20.0)
    kk = cen[rng.integers(0, 64, size=N)] + np.float32(0.004) * rng.standard_normal((N, H, d)).astype(np.float32)
    q, v = (rng.standard_normal((N, H, d)).astype(np.float32) for _ in range(2))
    return workloads.Workload("far_clusters", N, H, d, k, 0.25, None, workloads.bf16_round(q), workloads.bf16_round(kk),
                              workloads.bf16_round(v), None, False)


REAL = [
    # (kind, N, H, d, k)
    ("iid", 65549, 2, 16, 32), ("iid", 46007, 2, 32, 16), ("iid", 33001, 2, 64, 128),   # odd sizes of the key tree
    # two query blocks a wave: k <= 32 and ceil(N / 64) H >= 8192
    ("points", 65600, 8, 16, 32), ("points", 65600, 8, 16, 16), ("iid", 65600, 8, 16, 16),
    ("far", 65792, 2, 16, 32),
    ("iid", 200100, 1, 16, 200), ("iid", 200003, 1, 32, 400),                         # trees of 256 and 512 leaves
    ("iid", 65601, 1, 128, 100), ("iid", 33001, 2, 128, 40),                          # neither grouped nor bounded
]


@pytest.mark.parametrize("case", REAL, ids=lambda c: "%s_N%d_H%d_d%d_k%d" % c)
def test_sets_and_rows(case):
    kind, N, H, d, k = case
    if kind == "points":
        w = workloads.make(4, n=N, heads=H)
        w.k = k
    else:
        w = _far_clusters(N, H, d, k) if kind == "far" else workloads.iid(N, H, d, k, seed=N + d)
    assert (w.N, w.H, w.d) == (N, H, d)
    p = PathProbe(N, H, d, k)
    q, kk, v = _dev(w.q), _dev(w.kk), _dev(w.v)
    print(f"[case] streaming select {kind} N={N} H={H} d={d} k={k}", flush=True)
    out, idx, lse = kmip.fwd(q, kk, v, k, w.scale, workspace=p.ws)
    torch.cuda.synchronize()
    assert p.streamed()
    Qd, Kd, Vd = (oracle.from_bf16(a) for a in (w.q, w.kk, w.v))
    gi = idx.cpu().numpy()
    check_structure(gi, None, N, H, k)
    sel = stratified_rows(Qd, 8192, seed=123)
    exact, strict, loose = check_sets_all(w, Qd, Kd, gi, sel=sel)
    print(f"[sets] {exact} exact by scores, {strict} well-separated, {loose} near-tied of {len(sel)}", flush=True)
    ref_out, ref_lse = oracle.attend(Qd, Kd, Vd, gi, w.scale)
    allclose_report("out", out.cpu().numpy().reshape(-1, d), ref_out)
    allclose_report("lse", lse.cpu().numpy().reshape(-1), ref_lse)


# Small integers: scores are exact and tie everywhere, so the sampled rows are
# the oracle's index for index (score descending, index ascending).
@pytest.mark.parametrize("N,H,d,k", [(65600, 8, 16, 32), (65537, 2, 128, 32), (200001, 1, 16, 300), (200100, 1, 32, 512)],
                         ids=lambda x: str(x))
def test_integer_ties(N, H, d, k):
    rng = np.random.default_rng(N + d + k)
    qb = workloads.bf16_round(rng.integers(-2, 3, size=(N, H, d)).astype(np.float32))
    kb = workloads.bf16_round(rng.integers(-1, 2, size=(N, H, d)).astype(np.float32))
    p = PathProbe(N, H, d, k)
    print(f"[case] streaming select ties N={N} H={H} d={d} k={k}", flush=True)
    idx = kmip.topk(_dev(qb), _dev(kb), k, workspace=p.ws)
    torch.cuda.synchronize()
    assert p.streamed()
    gi = idx.cpu().numpy()
    check_structure(gi, None, N, H, k)
    sel = sample_rows(N, H, 512, seed=5)
    o_idx, _, _ = oracle.topk(oracle.from_bf16(qb), oracle.from_bf16(kb), k, sel=sel)
    np.testing.assert_array_equal(gi.reshape(N * H, k)[sel], o_idx)


@pytest.mark.parametrize("N,d,k", [(65600, 16, 32), (46500, 32, 16)])
def test_identical_keys(N, d, k):
    # every projection and every score of a query ties: keys 0 .. k-1, in order
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    q = torch.randn(N, 2, d, device=DEV, generator=g).bfloat16()
    kk = torch.randn(1, 2, d, device=DEV, generator=g).bfloat16().expand(N, 2, d).contiguous()
    p = PathProbe(N, 2, d, k)
    idx = kmip.topk(q, kk, k, workspace=p.ws)
    torch.cuda.synchronize()
    assert p.streamed()
    assert (idx == torch.arange(k, dtype=torch.int32, device=DEV)).all()


@pytest.mark.parametrize("dv,rate", [(16, 0.0), (64, 0.5)])
def test_aggregate_in_grouped_order(dv, rate):
    # the forward takes the aggregate in the grouped query order: the rows of
    # kmip_topk and kmip_attend, bit for bit, also with other value widths and
    # dropout, and the events in their order
    w = workloads.iid(66000, 2, 16, 16, seed=12, dv=dv)
    q, kk, v = _dev(w.q), _dev(w.kk), _dev(w.v)
    kw = {}
    if rate:
        keep = np.random.default_rng(1).random((w.N, w.H, w.k)) >= rate
        kw = dict(keep=torch.from_numpy(keep.astype(np.uint8)).to(DEV), drop_rate=rate)
    p = PathProbe(w.N, w.H, w.d, w.k)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    out, idx, lse = kmip.fwd(q, kk, v, w.k, w.scale, events=ev[:3], workspace=p.ws, **kw)
    ev[3].record()
    idx2 = kmip.topk(q, kk, w.k)
    out2, lse2 = kmip.attend(q, kk, v, idx2, w.scale, **kw)
    torch.cuda.synchronize()
    assert p.streamed()
    assert torch.equal(idx, idx2) and torch.equal(out, out2) and torch.equal(lse, lse2)
    assert ev[0].elapsed_time(ev[1]) > 0 and ev[1].elapsed_time(ev[2]) >= 0 and ev[2].elapsed_time(ev[3]) > 0
