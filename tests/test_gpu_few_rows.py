"""Saliency of at most 8 window rows (K read once, logits kept): row counts 1 to 8 on both
quads, sequences around the 16-key tiles and the chunks, chunks of up to 1024 keys (K rings past
their first fill), more sequences than the launch arguments hold, the causal tail, both head
dims, NaN and infinite keys, against the oracle, float64 and the two-sweep schedule. Both
schedules compute exp2(c z - lse) in fp32 with |c z - lse| below 64 here, so they differ by a few
roundings of that exponent: 64 * 2^-24 * ln 2 * 4 = 1.1e-5 at most. Against float64, a logit is
the fp32 sum of up to 128 exact products whose magnitudes sum to less than 12 after scaling
(unit normals: 128 * 0.64 / sqrt(128) = 7.2 on average), off by less than
128 * 2^-24 * 12 = 9.2e-5, and a row's LSE by no more: 2e-4 with the roundings above."""
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


RINGS = {
    # layers, KV heads, head dim, G, window, sequence lengths; the chunk these make
    "r1_d128_640": (4, 8, 128, 1, 1, [4100, 900]),
    "r3_d64_576": (3, 6, 64, 1, 3, [5000, 17, 3001]),
    "r5_d128_768": (2, 4, 128, 1, 5, [24333]),
    "r6_d64_1024": (8, 4, 64, 3, 2, [8200]),
    "r8_d128_1024": (16, 2, 128, 4, 2, [8207, 1, 0, 1030]),
}


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("case", list(RINGS))
def test_few_rows_long_chunks(case, causal):
    """Chunks of up to 16 tiles per wave, odd last chunks among them."""
    import torch

    from paper_2609_22158_amd import binding as B

    L, H, d, G, W, lens = RINGS[case]
    cu = np.concatenate([[0], np.cumsum(lens)])
    pb = B.Problem(L, H * G, H, d, W, cu, np.zeros(len(lens) + 1, np.int32))
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
            for s in ((L, len(lens), W, H * G, d), (L, H, int(cu[-1]), d)))
    log(f"[few rows {case} causal={causal}]")
    A = B.saliency(pb, q, k, B.Params(causal_tail=causal)).double()
    for s, n in enumerate(lens):
        a = int(cu[s])
        # rows (w, g) of every head: [L][H][W * G][d]
        rows = q[:, s].view(L, W, H, G, d).permute(0, 2, 1, 3, 4).reshape(L, H, W * G, d).double()
        z = (rows[:, :, :, None] * k[:, :, None, a:a + n].double()).sum(-1) / d ** 0.5
        if causal:
            last = n - W + torch.arange(W, device="cuda").repeat_interleave(G)
            z = z.masked_fill(torch.arange(n, device="cuda") > last[:, None], float("-inf"))
        p = torch.softmax(z, -1).nan_to_num(0.0)  # a row that sees no key adds nothing
        torch.testing.assert_close(A[:, :, a:a + n], p.sum(2), rtol=2e-4, atol=1e-30)


@pytest.mark.parametrize("bad", ["nan", "inf", "-inf"])
@pytest.mark.parametrize("d", [64, 128])
def test_few_rows_non_finite_keys(d, bad):
    """A key with a NaN or an infinity leaves NaN and finite values where two sweeps leave them."""
    import torch

    from paper_2609_22158_amd import binding as B

    lens = [1000, 17, 129]
    cu = np.concatenate([[0], np.cumsum(lens)])
    pb = B.Problem(1, 4, 1, d, 2, cu, np.zeros(len(lens) + 1, np.int32))
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
            for s in ((1, len(lens), 2, 4, d), (1, 1, int(cu[-1]), d)))
    for at in (333, 1016, 1100):  # inside, the last key of a sequence, inside
        k[0, 0, at, 5] = float(bad)
    out = [B.saliency(pb, q, k, B.Params(saliency_schedule=s)) for s in (0, 1)]
    assert bool(torch.isnan(out[0]).any())
    torch.testing.assert_close(out[0], out[1], rtol=1.1e-5, atol=1e-12, equal_nan=True)


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


def _random_cache(L, H, G, W, d, n, seed=7):
    import torch

    from paper_2609_22158_amd import binding as B

    gen = torch.Generator(device="cuda").manual_seed(seed)
    q, k = (torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
            for s in ((L, 1, W, H * G, d), (L, H, n, d)))
    steps = 20
    pb = B.Problem(L, H * G, H, d, W, np.array([0, n]), np.array([0, steps]))
    sid = (torch.arange(n, device="cuda") * steps // n).to(torch.int32)
    prot = (torch.arange(n, device="cuda") < 40).to(torch.uint8)
    util = torch.rand(steps, generator=gen, device="cuda")
    return pb, q, k, sid, prot, util


def test_workspace_of_a_wider_window_serves_few_rows():
    """A workspace sized for the same cache at window 64 has no room for logits: every entry point
    takes it and reads K twice, as the two-sweep schedule does."""
    import ctypes

    import torch

    from paper_2609_22158_amd import binding as B

    L, H, G, d, n, budget = 4, 4, 4, 128, 9000, 300
    lib = B.load()
    wide = B.Problem(L, H * G, H, d, 64, np.array([0, n]), np.array([0, 20]))
    size = {"saliency": wide.saliency_workspace_bytes(), "score": wide.workspace_bytes(),
            "compress": int(lib.stepkv_compress_workspace_bytes(ctypes.byref(wide.c))),
            "shared": int(lib.stepkv_score_shared_workspace_bytes(ctypes.byref(wide.c), 3))}
    pb, q, k, sid, prot, util = _random_cache(L, H, G, 1, d, n)
    assert size["saliency"] < pb.saliency_workspace_bytes()  # less than what holds the logits
    ws = {key: torch.empty(b, dtype=torch.uint8, device="cuda") for key, b in size.items()}
    rows = int(pb.retained_rows(prot.cpu().numpy(), budget)[-1])
    lse = B.window_lse(pb, q, k, workspace=ws["saliency"])
    res = {}
    for sched in (0, 1):
        prm = B.Params(saliency_schedule=sched)
        log(f"[few rows, workspace of window 64] schedule {sched}")
        out = [B.saliency(pb, q, k, prm, workspace=ws["saliency"]),
               B.saliency_from_lse(pb, q, k, lse, prm, workspace=ws["saliency"])]
        for kw in ({}, {"lse": lse}):
            out.append(B.score(pb, q, k, sid, prot, util, prm, workspace=ws["score"], **kw)["scores"])
            c = B.compress(pb, q, k, k, sid, prot, util, budget, rows, prm,
                           workspace=ws["compress"], **kw)
            out += [c["scores"], c["k_hat"]]
            out.append(B.score_shared(pb, q, k, sid, prot, util, prm, workspace=ws["shared"],
                                      **kw)["scores"])
        res[sched] = out
    for a, b in zip(res[0], res[1]):
        assert torch.equal(a, b)
    with pytest.raises(B.StepKVError):  # and still none below the sweeps' own need
        B.saliency(pb, q, k, workspace=ws["saliency"][:1024])
    ample = B.saliency(pb, q, k)  # the logits kept
    torch.testing.assert_close(ample, res[0][0], rtol=1.1e-5, atol=1e-12)


@pytest.mark.parametrize("G,n,groups", [(4, 32768, 2), (8, 32768, 3), (2, 6000, 1)])
def test_few_rows_in_groups_of_heads(G, n, groups):
    """32 layers x 8 heads: the logits in one group (a whole pass' workspace), in the groups that
    stepkv_saliency's own size makes and in those of the static scratch agree bit for bit."""
    import ctypes

    import torch

    from paper_2609_22158_amd import binding as B

    pb, q, k, sid, prot, util = _random_cache(32, 8, G, 1, 64, n)
    need, logits = pb.saliency_workspace_bytes(), 32 * 8 * n * 16 * (1 if G <= 4 else 2)
    assert need <= B.STATIC_SCRATCH_BYTES
    assert logits // groups <= need < logits // groups + (8 << 20)
    log(f"[few rows G={G} n={n}]")
    full = B.score(pb, q, k, sid, prot, util, want_saliency=True)
    A = B.saliency(pb, q, k)  # its own workspace size
    assert torch.equal(A, full["saliency"])
    scores, sal = torch.empty_like(A), torch.empty_like(A)
    rc = B.load().stepkv_score_noalloc(
        ctypes.byref(pb.c), ctypes.byref(B.Params().c()), q.data_ptr(), k.data_ptr(),
        sid.data_ptr(), prot.data_ptr(), util.data_ptr(), scores.data_ptr(), sal.data_ptr(), None,
        B._stream(None))
    assert rc == 0
    assert torch.equal(sal, A) and torch.equal(scores, full["scores"])
