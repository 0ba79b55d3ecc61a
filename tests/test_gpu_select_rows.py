"""Selection at the edges of its row paths: rows around 4096, 8192, 16384, 32768 and 65536
tokens (blocks of 4096 positions, register paths of 1 to 16 blocks, rows read again past 65536),
protected tokens anywhere in the row, budgets around 1024, 2048, 4096 and above (the bound on
tau from the m-th largest key per thread, m = 1, 2, 4, 8) and up to every candidate. Bit for bit
against the oracle's ranking of the same fp32 numbers."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_cases import log
from synth import make_workload
from tests.test_gpu_parity import _special_scores

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seqlens", [[1], [4095, 4096, 4097], [8191, 3, 8193], [16384, 16385],
                                     [32767, 32769], [65536], [65537, 5000], [98305]],
                         ids=lambda s: "-".join(map(str, s)))
def test_select_row_paths_bitexact(seqlens):
    import torch

    from paper_2609_22158_amd import binding as B

    w = make_workload("ragged16", seqlens=seqlens, num_layers=2, protected_len=0, with_v=False)
    pb = B.Problem.from_workload(w)
    P = _special_scores(w, 11)
    prot = (np.random.default_rng(5).random(w.total_tokens) < 0.02).astype(np.uint8)
    P[:, :, prot != 0] = -np.inf
    scores, pdev = torch.from_numpy(P).cuda(), torch.from_numpy(prot).cuda()
    sid = torch.from_numpy(w.step_ids).cuda()
    for budget in (1, 1023, 1025, 2049, 4097, 8200, 200000):
        log(f"[row paths {seqlens} B={budget}] gpu select")
        idx, cu, kept = B.select(pb, scores, pdev, sid, budget, want_kept=True)
        torch.cuda.synchronize()
        idx, cu, kept = idx.cpu().numpy(), cu.cpu().numpy(), kept.cpu().numpy()
        assert np.array_equal(cu, pb.retained_rows(prot, budget))
        for s in range(w.num_seqs):
            a, b = int(w.cu_seqlens[s]), int(w.cu_seqlens[s + 1])
            k0, k1 = int(w.cu_steps[s]), int(w.cu_steps[s + 1])
            free = prot[a:b] == 0
            for l in range(w.num_layers):
                for h in range(w.num_kv_heads):
                    with np.errstate(invalid="ignore"):
                        want = O.select_retained(P[l, h, a:b], free, budget)
                    got = idx[l, h, a:a + int(cu[s + 1] - cu[s])]
                    assert np.array_equal(got, want), (budget, s, l, h)
                    ids = w.step_ids[a:b][want[free[want]]]
                    assert np.array_equal(kept[l, h, k0:k1],
                                          np.bincount(ids[ids >= 0], minlength=k1 - k0))
