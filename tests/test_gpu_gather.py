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
# by head (wide rows, large k; a partly filled last workgroup per head)
CASES += [(1025, 3, 32, 32, 257), (1030, 2, 16, 16, 512), (1024, 3, 128, 128, 16), (1025, 3, 64, 64, 20)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "N%d_H%d_d%d_dv%d_k%d" % c)
def test_given_sets(case):
    N, H, d, dv, k = case
    rng = np.random.default_rng(d + dv + k)
    w = workloads.iid(N, H, d, min(k, N), seed=N + d + dv + k, dv=dv)
    # distinct keys per row where there are enough, random holes, a row without any
    idx = np.argsort(rng.random((N, H, N), dtype=np.float32), axis=2)[:, :, :k].astype(np.int32)
    idx = np.concatenate([idx, np.full((N, H, k - idx.shape[2]), -1, np.int32)], axis=2)
    holes = rng.random(idx.shape) < 0.1
    idx[0] = -1
    gpu_idx = np.where(holes, rng.choice(np.array([-1, -7, N, 2**31 - 1], np.int32), idx.shape), idx)
    ref_idx = np.where(holes, -1, idx)
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
    variants = [_lib.BWD_SEGMENTED] + ([_lib.BWD_BUCKETED] if d == dv <= 64 and k <= 128 else [])
    for variant in variants:
        got = kmip.bwd(q, kk, v, g, gi, lse, w.scale, variant=variant, **kw)
        for name, a, r in zip(("dQ", "dK", "dV"), got, grads):
            allclose_report(f"{name} v{variant}", a.cpu().numpy(), r)
