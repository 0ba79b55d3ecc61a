"""The one-launch priority and selection of stepkv_compress against stepkv_score and
stepkv_select, bit for bit: row lengths around the waves' 256 positions and the blocks of 4096,
pooling windows 1 to 9 (in registers) and 11 (the separate kernels), protected tokens and
out-of-range step ids anywhere, a NaN key, and the status word's flags; the same without a
status word; and step counts around the table that it keeps in LDS."""
import numpy as np
import pytest

from tests.gpu_cases import gpu_utilities, log
from synth import make_workload

pytestmark = pytest.mark.gpu

LENGTHS = {"short": [1, 0, 3, 255, 256, 257, 1000], "block": [4095, 4096, 4097, 8191],
           "blocks": [8192, 8193, 16384], "rows": [16385, 32768, 5]}


@pytest.mark.parametrize("pool", [1, 3, 5, 7, 9, 11])
@pytest.mark.parametrize("lengths", list(LENGTHS))
def test_compress_equals_score_and_select(lengths, pool):
    import torch

    from paper_2609_22158_amd import binding as B

    w = make_workload("ragged16", seqlens=LENGTHS[lengths], num_layers=2, protected_len=0,
                      budget=700)
    pb = B.Problem.from_workload(w)
    rng = np.random.default_rng(pool)
    prot = (rng.random(w.total_tokens) < 0.03).astype(np.uint8)
    ids = w.step_ids.copy()
    ids[rng.random(w.total_tokens) < 0.001] = 1 << 20
    ids[rng.random(w.total_tokens) < 0.001] = -7
    kk = w.k.copy()
    if pool == 3:
        kk[0, 0, w.total_tokens // 2] = 0x7FC0  # a NaN key in one row
    q, k, v = (B.bf16_from_bits(x) for x in (w.q_win, kk, w.v))
    sid, pdev = torch.from_numpy(ids).cuda(), torch.from_numpy(prot).cuda()
    util = torch.from_numpy(gpu_utilities(w)).cuda()
    prm = B.Params(pool_kernel=pool, alpha=0.7, beta=0.3)
    rows = int(pb.retained_rows(prot, w.budget)[-1])
    log(f"[rank {lengths} pool={pool}] score and select")
    P = B.score(pb, q, k, sid, pdev, util, prm)["scores"]
    idx, cu, _ = B.select(pb, P, pdev, sid, w.budget)
    flags = pb.status(clear=True)
    log(f"[rank {lengths} pool={pool}] compress")
    res = B.compress(pb, q, k, v, sid, pdev, util, w.budget, rows, prm)
    assert pb.status(clear=True) == flags
    assert bool(flags & B.FLAG_NONFINITE) == (pool == 3)
    assert np.array_equal(res["scores"].cpu().numpy().view(np.uint32), P.cpu().numpy().view(np.uint32))
    assert np.array_equal(res["cu_retained"].cpu().numpy(), cu.cpu().numpy())
    quiet = B.Problem.from_workload(w, status=False)  # code of its own, without the flags
    log(f"[rank {lengths} pool={pool}] compress without a status word")
    other = B.compress(quiet, q, k, v, sid, pdev, util, w.budget, rows, prm)
    for key in ("scores", "cu_retained"):
        assert torch.equal(other[key].view(torch.int32), res[key].view(torch.int32)), key
    c, got, want = cu.cpu().numpy(), res["idx"].cpu().numpy(), idx.cpu().numpy()
    bare = other["idx"].cpu().numpy()
    for s in range(w.num_seqs):
        a = int(w.cu_seqlens[s])
        n = int(c[s + 1] - c[s])
        assert np.array_equal(got[:, :, a:a + n], want[:, :, a:a + n])
        assert np.array_equal(bare[:, :, a:a + n], want[:, :, a:a + n])


@pytest.mark.parametrize("steps", [0, 1, 4096, 4097])
def test_compress_step_counts(steps):
    """Steps in a sequence up to 4096 (the ranking's table of utilities) and one more (the
    separate kernels), and none at all."""
    import torch

    from paper_2609_22158_amd import binding as B

    n, L, H = 9001, 2, 2
    gen = torch.Generator(device="cuda").manual_seed(steps)
    q, k = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
            for s in ((L, 1, 16, 4 * H, 128), (L, H, n, 128)))
    pb = B.Problem(L, 4 * H, H, 128, 16, np.array([0, n]), np.array([0, steps]))
    # every step id occurs, the last one among them
    sid = (torch.arange(n, device="cuda") * max(steps, 1) // n).to(torch.int32)
    prot = (torch.arange(n, device="cuda") % 37 == 0).to(torch.uint8)
    util = torch.rand(steps, generator=gen, device="cuda")
    rows = int(pb.retained_rows(prot.cpu().numpy(), 500)[-1])
    log(f"[rank {steps} steps]")
    P = B.score(pb, q, k, sid, prot, util)["scores"]
    idx, cu, _ = B.select(pb, P, prot, sid, 500)
    res = B.compress(pb, q, k, k, sid, prot, util, 500, rows)
    assert bool(pb.status() & B.FLAG_STEP_ID) == (steps == 0)
    assert torch.equal(res["scores"], P) and torch.equal(res["cu_retained"], cu)
    assert torch.equal(res["idx"][:, :, :rows], idx[:, :, :rows])


@pytest.mark.parametrize("bits", [0x7FC00000, 0xFFFFFFFF, 0xFFC00001])
def test_compress_from_nan_lse(bits):
    """A NaN row LSE of any payload leaves NaN priorities (ranked as -inf, flagged), never a
    token that counts as protected."""
    import torch

    from paper_2609_22158_amd import binding as B

    w = make_workload("l1_8k", seqlens=[3000, 5000], num_layers=1, protected_len=0, budget=300)
    pb = B.Problem.from_workload(w)
    q, k, v = (B.bf16_from_bits(x) for x in (w.q_win, w.k, w.v))
    rng = np.random.default_rng(1)
    prot = (rng.random(w.total_tokens) < 0.03).astype(np.uint8)
    sid, pdev = torch.from_numpy(w.step_ids).cuda(), torch.from_numpy(prot).cuda()
    util = torch.from_numpy(gpu_utilities(w)).cuda()
    lse = B.window_lse(pb, q, k)
    lse.view(torch.int32)[0, 0, 5, 0] = bits - (1 << 32) if bits >> 31 else bits  # head 0
    pb.status(clear=True)
    log(f"[rank NaN lse {bits:#x}]")
    P = B.score(pb, q, k, sid, pdev, util, lse=lse)["scores"]
    idx, cu, _ = B.select(pb, P, pdev, sid, w.budget)
    flags = pb.status(clear=True)
    res = B.compress(pb, q, k, v, sid, pdev, util, w.budget, w.total_tokens, lse=lse)
    assert flags & B.FLAG_NONFINITE and pb.status(clear=True) == flags
    assert torch.equal(res["cu_retained"], cu)
    # NaN payloads may differ between the kernels, so NaN as NaN, everything else bit for bit
    nan = torch.isnan(P)
    assert bool(nan.any()) and torch.equal(torch.isnan(res["scores"]), nan)
    assert torch.equal(res["scores"].masked_fill(nan, 0.0), P.masked_fill(nan, 0.0))
    for s in range(w.num_seqs):
        a, n = int(w.cu_seqlens[s]), int(cu[s + 1] - cu[s])
        assert torch.equal(res["idx"][:, :, a:a + n], idx[:, :, a:a + n])
