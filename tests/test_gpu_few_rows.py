"""Saliency of at most 8 window rows (K read once, logits kept): row counts 1 to 8 on both
quads, sequences around the 16-key tiles and the chunks, more sequences than the launch
arguments hold, the causal tail and both head dims, against the oracle and against the
two-sweep schedule. Both sides compute exp2(c z - lse) in fp32 with |c z - lse| below 64 here,
so they differ by a few roundings of that exponent: 64 * 2^-24 * ln 2 * 4 = 1.1e-5 at most."""
import numpy as np
import pytest

import oracle as O
from synth import make_workload
from tests.gpu_cases import SCORE_RTOL, log

pytestmark = pytest.mark.gpu

SHAPES = {
    # name, window, sequence lengths
    "w1_g2_d64": ("tiny", 1, [1024]),
    "w4_g2_d64": ("tiny", 4, [1, 0, 15, 16, 17, 63, 1025, 129]),
    "w1_g4": ("l1_8k", 1, [4099]),
    "w2_g4": ("l1_8k", 2, [5, 2048, 1]),
    "w1_g7": ("ragged16", 1, [700, 16, 33]),
    "w1_g4_many": ("l1_8k", 1, [7 + 5 * i for i in range(40)]),
}


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_few_rows_saliency(shape, causal):
    import torch

    from paper_2609_22158_amd import binding as B

    name, window, lens = SHAPES[shape]
    w = make_workload(name, seqlens=lens, num_layers=2, window=window, protected_len=0,
                      with_v=False)
    pb = B.Problem.from_workload(w)
    q, k = B.bf16_from_bits(w.q_win), B.bf16_from_bits(w.k)
    out = {}
    for sched in (0, 1):
        log(f"[few rows {shape} causal={causal}] schedule {sched}")
        out[sched] = B.saliency(pb, q, k, B.Params(causal_tail=causal, saliency_schedule=sched))
    torch.cuda.synchronize()
    A = out[0].cpu().numpy()
    np.testing.assert_allclose(A, out[1].cpu().numpy(), rtol=1.1e-5, atol=1e-12)
    G = w.group
    for l in range(w.num_layers):
        for h in range(w.num_kv_heads):
            for s in range(w.num_seqs):
                a, b = int(w.cu_seqlens[s]), int(w.cu_seqlens[s + 1])
                if b == a:
                    continue
                rows = O.window_rows(O.decode_bf16(w.q_win[l, s]), h, G)
                vis = O.visible_keys(b - a, window, G, bool(causal))
                ref = O.window_saliency(rows, O.decode_bf16(w.k[l, h, a:b]),
                                        1.0 / np.sqrt(w.head_dim), vis)
                np.testing.assert_allclose(A[l, h, a:b], ref, rtol=SCORE_RTOL, atol=1e-9)


def test_few_rows_workspace_stays_in_bounds():
    """The logits of the last tile of every sequence stay inside the declared workspace."""
    import torch

    from paper_2609_22158_amd import binding as B

    w = make_workload("ragged16", seqlens=[1, 17, 0, 31, 2000], num_layers=2, window=1,
                      protected_len=0, with_v=False)
    pb = B.Problem.from_workload(w)
    q, k = B.bf16_from_bits(w.q_win), B.bf16_from_bits(w.k)
    need = pb.saliency_workspace_bytes()
    ws = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    B.saliency(pb, q, k, B.Params(), workspace=ws[:need])
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xA5).all())


def test_long_sequence_is_not_slower_than_two_sweeps():
    """One head of 524288 keys. Every workgroup of the sums reads all partials of its sequence,
    so short chunks cost the square of their number: 125 us with chunks of 192 keys, 57 with two
    sweeps, 40 with chunks of 1024."""
    import torch

    from paper_2609_22158_amd import binding as B

    n = 524288
    pb = B.Problem(1, 4, 1, 128, 1, np.array([0, n]), np.zeros(2, np.int32))
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
            for s in ((1, 1, 1, 4, 128), (1, 1, n, 128)))
    ws = torch.empty(pb.saliency_workspace_bytes(), dtype=torch.uint8, device="cuda")
    out = {s: torch.empty((1, 1, n), device="cuda") for s in (0, 1)}

    def passes(sched):  # ms of 20 passes
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            B.saliency(pb, q, k, B.Params(saliency_schedule=sched), workspace=ws, out=out[sched])
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b)

    log("[few rows long]")
    t = {s: sorted(passes(s) for _ in range(5))[2] for s in (0, 1)}
    torch.testing.assert_close(out[0], out[1], rtol=1.1e-5, atol=1e-12)
    assert t[0] < 1.3 * t[1], t
