"""The row gathers (aggregate and the sorted backward variants) on given index
sets, against the oracle: every pair of row widths, k at the edges of the
16-slot rounds, empty and out-of-range slots, dropout, both orders of the
query-heads."""
import numpy as np
import pytest

import oracle
import workloads
from parity import allclose_report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2604_03815_amd as kmip  # noqa: E402
from paper_2604_03815_amd import _lib  # noqa: E402

DEV = torch.device("cuda:0")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).to(DEV)


CASES = [(70, 2, d, dv, k) for d, dv, k in (
    (16, 16, 1), (16, 16, 17), (16, 32, 16), (16, 64, 33), (16, 128, 128), (32, 16, 15), (32, 32, 16), (32, 32, 65),
    (32, 64, 32), (32, 128, 8), (64, 16, 129), (64, 32, 17), (64, 64, 1), (64, 64, 128), (64, 128, 31), (128, 16, 5),
    (128, 32, 128), (128, 64, 16), (128, 128, 33))]
# more than 2^20 pairs at d = 128 and k > 128, 2^16 at unequal widths: the bucketed
# reduction's forms for them (k up to 256 and 512: 8 and 4 teams a workgroup)
CASES += [(3001, 3, 128, 128, 128), (2100, 2, 32, 64, 16), (2051, 3, 64, 16, 20), (2060, 1, 16, 128, 40), (2050, 2, 32, 32, 300), (2100, 4, 64, 64, 129), (4099, 2, 16, 16, 512)]
# several pieces of 4096 pairs a bucket, row groups of 4 to 32 lanes, some of them idle
CASES += [(2060, 1, 16, 16, 40), (2060, 1, 16, 32, 40), (2060, 1, 32, 16, 64), (2060, 1, 16, 64, 33), (2060, 1, 64, 32, 128), (2060, 1, 64, 128, 100), (2060, 1, 128, 64, 128)]
# by head (wide rows, large k; a partly filled last workgroup per head)
CASES += [(1025, 3, 32, 32, 257), (1030, 2, 16, 16, 512), (1024, 3, 128, 128, 16), (1025, 3, 64, 64, 20)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%d_H%d_d%d_dv%d_k%d" % c)
def test_given_sets(case):
    N, H, d, dv, k = case
    rng = np.random.default_rng(d + dv + k)
    w = workloads.iid(N, H, d, min(k, N), seed=N + d + dv + k, dv=dv)
    # distinct keys per row where there are enough, random holes, a row without any
    if N > 2000:   # (a stride coprime to a prime modulus above N keeps a row's keys distinct)
        step = rng.integers(1, 4799, (N, H, 1))
        idx = ((rng.integers(0, 4799, (N, H, 1)) + step * np.arange(k)) % 4799).astype(np.int32)
        idx[idx >= N] = -1
    else:
        idx = np.argsort(rng.random((N, H, N), dtype=np.float32), axis=2)[:, :, :k].astype(np.int32)
        idx = np.concatenate([idx, np.full((N, H, k - idx.shape[2]), -1, np.int32)], axis=2)
    holes = rng.random(idx.shape) < 0.1
    idx[0] = -1
    gpu_idx = np.where(holes, rng.choice(np.array([-1, -7, N, 2**31 - 1], np.int32), idx.shape), idx)
    ref_idx = np.where(holes, -1, idx)
    assert ((np.sort(ref_idx, 2)[:, :, 1:] != np.sort(ref_idx, 2)[:, :, :-1]) | (np.sort(ref_idx, 2)[:, :, 1:] < 0)).all()
    rate = 0.25 if k % 2 else 0.0
    keep = (rng.random(idx.shape) >= rate).astype(np.uint8) if rate else None
    kw = {} if keep is None else dict(keep=torch.from_numpy(keep).to(DEV), drop_rate=rate)
    okw = {} if keep is None else dict(keep=keep, drop_rate=rate)
    print(f"[case] gather N={N} H={H} d={d} dv={dv} k={k} rate={rate}", flush=True)
    q, kk, v, g = _dev(w.q), _dev(w.kk), _dev(w.v), _dev(w.dout)
    gi = torch.from_numpy(np.ascontiguousarray(gpu_idx)).to(DEV)
    Qd, Kd, Vd, Gd = (oracle.from_bf16(a) for a in (w.q, w.kk, w.v, w.dout))
    out, lse = kmip.attend(q, kk, v, gi, w.scale, **kw)
    ro, rl = oracle.attend(Qd, Kd, Vd, ref_idx, w.scale, **okw)
    allclose_report("out", out.cpu().numpy().reshape(-1, dv), ro)
    allclose_report("lse", lse.cpu().numpy().reshape(-1), rl)
    grads = oracle.backward(Qd, Kd, Vd, Gd, ref_idx, w.scale, **okw)
    variants = [_lib.BWD_AUTO, _lib.BWD_SEGMENTED] + ([_lib.BWD_BUCKETED] if d == dv <= 64 and k <= 128 else [])
    for variant in variants:
        got = kmip.bwd(q, kk, v, g, gi, lse, w.scale, variant=variant, **kw)
        for name, a, r in zip(("dQ", "dK", "dV"), got, grads):
            allclose_report(f"{name} v{variant}", a.cpu().numpy(), r)


@pytest.mark.parametrize("N,d,dv,k", [
    (14, 16, 16, 4), (12, 64, 128, 3), (16, 16, 32, 5), (24, 128, 16, 9), (40, 32, 64, 17),
    # up to 6144 query-heads (12288 past k = 128), four teams share one where k > 32; 64 slots a round past k = 256 up to N (d + d_V) = 5 2^18
    (70, 64, 32, 33), (134, 32, 32, 64), (86, 128, 128, 40), (520, 16, 16, 257), (806, 64, 64, 400), (3072, 16, 64, 100),
    (3073, 16, 64, 100), (3100, 32, 32, 64), (6144, 32, 64, 129), (6145, 32, 64, 129), (6150, 16, 32, 300), (6150, 32, 16, 512),
    (6150, 64, 16, 257)])
def test_rows_that_end_early(N, d, dv, k):
    # the aggregate looks at a row's slots up to the last one kept, a few, 16 or
    # 64 at a time: rows that keep their first 0, 1, .. slots, with holes
    H = 2
    rng = np.random.default_rng(d + dv + k)
    w = workloads.iid(N, H, d, k, seed=d + dv + k, dv=dv)
    step = np.array([s for s in range(1, N) if np.gcd(s, N) == 1])   # distinct keys in a row
    idx = ((rng.integers(0, N, (N, H, 1)) + rng.choice(step, (N, H, 1)) * np.arange(k)) % N).astype(np.int32)
    idx[np.arange(k) >= (np.arange(N) % (k + 1))[:, None, None] + np.zeros((N, H, 1), int)] = -1
    idx[rng.random(idx.shape) < 0.1] = -1
    keep = (rng.random(idx.shape) >= 0.25).astype(np.uint8)
    print(f"[case] gather, short rows N={N} d={d} dv={dv} k={k}", flush=True)
    q, kk, v = _dev(w.q), _dev(w.kk), _dev(w.v)
    out, lse = kmip.attend(q, kk, v, torch.from_numpy(idx).to(DEV), w.scale, keep=torch.from_numpy(keep).to(DEV), drop_rate=0.25)
    ro, rl = oracle.attend(*(oracle.from_bf16(a) for a in (w.q, w.kk, w.v)), idx, w.scale, keep=keep, drop_rate=0.25)
    allclose_report("out", out.cpu().numpy().reshape(-1, dv), ro)
    allclose_report("lse", lse.cpu().numpy().reshape(-1), rl)


def test_key_sort_workspace_still_taken():
    # a workspace that holds only the key sort's arrays gets the key sort
    N, H, d, dv, k = 3000, 2, 32, 64, 16
    w = workloads.iid(N, H, d, k, seed=5, dv=dv)
    q, kk, v, g = _dev(w.q), _dev(w.kk), _dev(w.v), _dev(w.dout)
    small = kmip.bwd_workspace_size(N, H, d, k, _lib.BWD_SEGMENTED, dv=dv)
    assert small < kmip.bwd_workspace_size(N, H, d, k, _lib.BWD_AUTO, dv=dv)
    out, idx, lse = kmip.fwd(q, kk, v, k, w.scale)
    buf = torch.empty(small, dtype=torch.uint8, device=DEV)
    got = [torch.empty(N, H, x, device=DEV) for x in (d, d, dv)]
    _lib.check(_lib.load().kmip_bwd_ex(q.data_ptr(), kk.data_ptr(), v.data_ptr(), g.data_ptr(), idx.data_ptr(), lse.data_ptr(),
                                       None, 0.0, N, H, d, dv, k, w.scale, *(t.data_ptr() for t in got), _lib.BWD_AUTO,
                                       buf.data_ptr(), small, torch.cuda.current_stream().cuda_stream))
    want = kmip.bwd(q, kk, v, g, idx, lse, w.scale)
    for name, a, b in zip(("dQ", "dK", "dV"), got, want):
        allclose_report(name, a.cpu().numpy(), b.cpu().numpy(), atol=1e-5, rtol=1e-4)   # 32-bit sums in another order
