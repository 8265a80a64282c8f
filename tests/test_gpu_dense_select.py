"""The dense select (scores in registers, or two passes over the keys) and the
lines at which the library changes path, against the oracle.

Integer inputs: the fp32 scores are exact and tie everywhere, so every row
must equal the oracle's, order (score descending, index ascending) included.
"""
import numpy as np
import pytest

import oracle
import workloads
from parity import check_structure, sample_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2604_03815_amd as kmip  # noqa: E402

DEV = torch.device("cuda:0")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(DEV)


EDGES = [1, 31, 32, 33, 0, 480, 511, 512, 513, 700]   # tiles, and the 512-key register path
BIG = [257, 288, 300, 320, 385, 460, 512]             # more nodes than a list of 256 keys takes
CASES = [
    # (N, H, d, k, sizes, inputs)
    *[(sum(EDGES), 2, d, k, EDGES, "ints") for d, k in ((16, 1), (32, 32), (64, 33), (128, 16), (128, 128), (32, 128))],
    *[(2733, 1, 32, k, [600, 31, 2, 2100], "ints") for k in (129, 256, 257, 512)],
    # graphs of few groups per kept key: four rows a group, pairs
    *[(sum(BIG), 2, d, k, BIG, "ints") for d, k in ((32, 64), (16, 80), (32, 100), (64, 103), (128, 112))],
    (512, 3, 32, 16, None, "ints"),
    (513, 3, 32, 16, None, "ints"),
    # lists that overflow: zero queries (every key ties), keys in order of score
    *[(3000, 1, 32, k, s, kind) for k, s in ((10, None), (128, [500, 2500]), (300, None)) for kind in ("zeros", "sorted")],
    # few distinct keys: ties at every query's k-th best, listed again up to the bound
    (9000, 2, 128, 32, None, "copies"),
    (4000, 1, 64, 100, [1500, 2500], "copies"),
    (31000, 1, 16, 16, None, "copies"),
    (2600, 1, 32, 300, None, "copies"),
    # ties in lists of more than 128 keys: all keys, a few scores, all but one
    *[(sum(EDGES), 2, d, k, EDGES, kind) for d, k, kind in
      ((32, 64, "zeros"), (16, 100, "zeros"), (64, 128, "zeros"), (32, 100, "spike"), (16, 64, "copies"))],
    *[(2600, 1, 32, k, s, "spike") for k, s in ((40, None), (128, [900, 1700]), (200, None), (512, None))],
    # clusters one after the other: a query's best keys fill few tiles
    (9000, 2, 32, 16, None, "runs"),
    (45000, 1, 32, 16, None, "runs"),
    (12000, 2, 64, 128, [5000, 7000], "runs"),
    (12000, 1, 16, 200, None, "runs"),
    (12000, 1, 16, 512, None, "runs"),
    # 64 queries a task; sampled first passes (every second, every third tile)
    (31000, 1, 16, 32, None, "ints"),
    (42000, 1, 16, 10, None, "ints"),
    (16500, 1, 64, 4, None, "ints"),
    (12000, 1, 64, 16, [400, 11600], "ints"),
    # the last size of the dense path and the first of the streaming kernel
    (46000, 1, 32, 16, None, "ints"),
    (46001, 1, 32, 16, None, "ints"),
    (65537, 1, 16, 10, None, "ints"),
    (65700, 1, 16, 16, [100, 65600], "ints"),
    (200001, 1, 16, 130, None, "ints"),
    # wide keys, 32 < k < 64: a graph on either side of the line in one batch
    (65600, 1, 64, 40, [32768, 32769, 63], "ints"),
    (33200, 2, 128, 33, [400, 32800], "ints"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%d_H%d_d%d_k%d_G%s_%s" % (*c[:4], c[4] and len(c[4]), c[5]))
def test_rows_equal_oracle(case):
    N, H, d, k, sizes, kind = case
    rng = np.random.default_rng(N + d + k)
    q = rng.integers(-2, 3, size=(N, H, d)).astype(np.float32)
    kk = rng.integers(-1, 2, size=(N, H, d)).astype(np.float32)
    if kind == "zeros":
        q[rng.random(N) < 0.5] = 0
    elif kind == "spike":
        kk[:] = np.where(rng.random((N, 1, 1)) < 0.01, rng.integers(1, 100, (N, 1, 1)), 0)
        q = np.abs(q) + 1
    elif kind == "copies":
        kk = kk[rng.integers(0, 50, N)]
    elif kind == "runs":
        kk += rng.integers(-8, 9, size=(40, H, d))[np.sort(rng.integers(0, 40, N))]
    elif kind == "sorted":
        q[:] = 1
        kk[:] = 0
        kk[:, :, 0] = np.minimum(np.arange(N) // 12, 255)[:, None]   # exact in bf16, twelve keys a score
    offsets = None if sizes is None else np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    qb, kb = workloads.bf16_round(q), workloads.bf16_round(kk)
    print(f"[case] dense select N={N} H={H} d={d} k={k} sizes={sizes} {kind}", flush=True)
    idx = kmip.topk(_dev(qb), _dev(kb), k, graph_offsets=offsets)
    torch.cuda.synchronize()
    idx = idx.cpu().numpy()
    check_structure(idx, offsets, N, H, k)
    sel = None if N * H <= 8000 else sample_rows(N, H, 512, seed=5)
    o_idx, _, _ = oracle.topk(oracle.from_bf16(qb), oracle.from_bf16(kb), k, offsets=offsets, **({} if sel is None else {"sel": sel}))
    got = idx.reshape(N * H, k)
    np.testing.assert_array_equal(got if sel is None else got[sel], o_idx)


# Inputs whose lists overflow at every listing, so that the block walks the
# tiles one at a time.  The good keys all lie in the first rows of every eighth
# tile (sixteenth for k > 128): a handful of group maxima holds them, so the
# threshold lies below all of them, and one wave lists them in rising order, so
# a list of CAP keys raises the bound past CAP - k of them only.
WALK = [
    # (d, k, sizes, CAP); the walked graph is the largest
    (16, 32, [28000], 128),            # 32 queries a block
    (16, 32, [60000], 128),            # 64 queries a block
    (128, 16, [24000], 128),           # sampled first pass
    (32, 30, [33, 40000, 20], 128),    # a batch, the graph's first tile shared with another
    (16, 128, [50000], 256),
    (16, 256, [140000], 512),
    (16, 512, [140000], 1024),         # 16 queries a block
]


@pytest.mark.parametrize("case", WALK, ids=lambda c: "d%d_k%d_N%d_G%d" % (c[0], c[1], sum(c[2]), len(c[2])))
def test_tile_by_tile_walk(case):
    d, k, sizes, cap = case
    rng = np.random.default_rng(d + k)
    N, big = sum(sizes), int(np.argmax(sizes))
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    lo, hi = int(offsets[big]), int(offsets[big + 1])
    at = np.arange(N) - (lo & ~31)                 # row from the graph's first tile
    period, rows = {128: (256, 4), 256: (256, 4), 512: (512, 4), 1024: (512, 8)}[cap]
    good = (np.arange(N) >= lo) & (np.arange(N) < hi) & (at % period < rows)
    M = int(good.sum())
    assert M - 2 * (cap - k) > cap, "three listings overflow"
    # scores 256 a + b of a query (256, 1, 0, ..): exact, the good ones rising
    # and above all others
    val = rng.integers(0, 25600, size=N)
    val[good] = 51200 + np.arange(M)
    kk = np.zeros((N, 1, d), np.float32)
    kk[:, 0, 0], kk[:, 0, 1] = val // 256, val % 256
    q = np.zeros((N, 1, d), np.float32)
    q[:, 0, 0], q[:, 0, 1] = 256, 1
    kind = rng.random(N)
    q[kind < 0.2] *= -1                            # the lowest keys win
    q[kind > 0.95] = 0                             # every key ties
    qb, kb = workloads.bf16_round(q), workloads.bf16_round(kk)
    print(f"[case] dense select walk N={N} d={d} k={k} sizes={sizes}", flush=True)
    off = None if len(sizes) == 1 else offsets
    idx = kmip.topk(_dev(qb), _dev(kb), k, graph_offsets=off)
    torch.cuda.synchronize()
    idx = idx.cpu().numpy()
    check_structure(idx, off, N, 1, k)
    got = idx.reshape(N, k)
    up = (kind >= 0.2) & (kind <= 0.95) & (np.arange(N) >= lo) & (np.arange(N) < hi)
    want = np.nonzero(good)[0][::-1][:k]
    assert (got[up] == want).all(), "rows of the queries whose lists overflow"
    sel = sample_rows(N, 1, 512, seed=5)
    o_idx, _, _ = oracle.topk(oracle.from_bf16(qb), oracle.from_bf16(kb), k, offsets=off, sel=sel)
    np.testing.assert_array_equal(got[sel], o_idx)


def test_more_blocks_than_a_launch_holds():
    # Graphs of two nodes (one and none among them) with many heads: more
    # workgroups than one launch of 2^31 threads, so the last heads come from
    # a second launch.  Small integers: scores are exact and tie.
    H, d, k = 66000, 16, 2
    sizes = [2] * 60 + [1, 0] * 5
    N = sum(sizes)
    assert sum(s > 0 for s in sizes) * H * 512 > 2**31
    gen = torch.Generator(device=DEV)
    gen.manual_seed(63)
    q, kk = (torch.randint(-2, 3, (N, H, d), generator=gen, device=DEV, dtype=torch.int8).to(torch.bfloat16) for _ in range(2))
    print(f"[case] dense select slices N={N} H={H} d={d} k={k}", flush=True)
    idx = kmip.topk(q, kk, k, graph_offsets=np.concatenate([[0], np.cumsum(sizes)]))
    torch.cuda.synchronize()
    a = torch.arange(0, 120, 2, device=DEV)
    for i in (0, 1):
        s = [(q[a + i].float() * kk[a + j].float()).sum(-1) for j in (0, 1)]
        first = torch.where(s[0] >= s[1], 0, 1) + a[:, None]
        assert torch.equal(idx[a + i, :, 0], first.int())
        assert torch.equal(idx[a + i, :, 1], (2 * a[:, None] + 1 - first).int())
    one = torch.arange(120, N, device=DEV)
    assert (idx[one, :, 0] == one[:, None]).all() and (idx[one, :, 1] == -1).all()
