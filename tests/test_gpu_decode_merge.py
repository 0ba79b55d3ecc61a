"""Decode: splits shared by 4, 8 and 16 waves and the four forms of the merge (all heads of a
KV head per workgroup of 128 or 256 threads; one head with one or several thread groups over the
splits), each with one split, a few and more than 64 per sequence, empty and one-row sequences, an
out_rows that cuts the last one, and NaN and infinite rows.
P enters the second product as two bf16 parts (2^-17 relative) and every sum is fp32, so an
output differs from float64 attention by less than 2^-15 of its row's largest magnitude."""
import numpy as np
import pytest

from tests.gpu_cases import log

pytestmark = pytest.mark.gpu

CASES = {
    # layers, q heads, kv heads, d, rows per sequence, rows cut off the end
    "waves8": (1, 32, 8, 128, [1536], 0),
    "waves16_edges": (1, 8, 2, 64, [63, 64, 65, 0, 1, 127], 0),
    "waves8_many": (1, 4, 1, 128, [9000], 100),
    "waves4_many_splits": (2, 14, 2, 64, [40000, 5], 0),
    "one_head_128": (16, 64, 8, 128, [300, 77], 0),
    "all_heads": (16, 28, 4, 64, [100, 600, 0, 1300, 64, 1, 900, 513], 300),
    "all_heads_split1024": (32, 16, 8, 64, [7000, 1, 300], 0),
    # kv heads x sequences >= 512: all heads per workgroup, 79 splits in one sequence
    "all_heads_many_splits": (1, 7, 1, 64, [3, 40000, 2600] + [0, 1, 17] * 180, 0),
    "all_heads_many_splits_d128": (2, 6, 2, 128, [33300, 700] + [0, 5] * 90, 3),
    # fewer, but 1024 query heads: 128 threads per head; 1, 6 and 79 splits
    "one_head_128_splits": (1, 8, 1, 64, [3000, 40000, 1] + [0, 20] * 70, 0),
    "one_head_128_splits_d128": (2, 64, 4, 128, [2700, 33300] + [0, 9] * 10, 5),
    # at least 64 rows a sequence on average: 16 waves at d 64
    "waves16_edges_64_rows": (1, 8, 2, 64, [63, 64, 65, 0, 1, 127, 200], 1),
    # few splits a sequence on average, (head, dim) pairs for 256 or 128 threads
    "few_all_heads_256": (1, 8, 2, 64, [33300, 700] + [0, 5, 513] * 20, 3),
    "few_all_heads_128": (1, 2, 2, 64, [3, 40000, 2600] + [0, 1, 17] * 30, 0),
    "few_all_heads_128_d128": (4, 8, 8, 128, [512, 1], 0),
    # kv heads x sequences >= 512: 128 threads for two heads of d 64, one head each of G 1
    "all_heads_128_splits": (2, 8, 4, 64, [40000, 2600] + [0, 1, 17] * 30, 0),
    "one_of_one_head": (1, 4, 4, 128, [33300, 2600] + [0, 5, 600] * 50, 2),
}


@pytest.mark.parametrize("case", list(CASES))
def test_decode_merge(case):
    import torch

    from paper_2609_22158_amd import binding as B

    L, Hq, Hkv, d, rows, cut = CASES[case]
    S, G = len(rows), Hq // Hkv
    cu = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    out_rows = int(cu[-1]) - cut
    # sequences longer than what they retain, as after compaction
    pb = B.Problem(L, Hq, Hkv, d, 1, np.concatenate([[0], np.cumsum([r + 50 for r in rows])]),
                   np.zeros(S + 1, np.int32))
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = torch.randn((L, S, Hq, d), generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn((L, Hkv, out_rows, d), generator=gen, device="cuda").to(torch.bfloat16)
    v = torch.randn((L, Hkv, out_rows, d), generator=gen, device="cuda").to(torch.bfloat16)
    log(f"[decode merge {case}]")
    out = B.decode_attention(pb, q, k, v, torch.from_numpy(cu).cuda(), out_rows)
    torch.cuda.synchronize()
    assert bool(pb.status() & B.FLAG_OUT_ROWS) == (cut > 0)
    q, k, v, out = q.double(), k.double(), v.double(), out.double()
    for s in range(S):
        a, b = min(int(cu[s]), out_rows), min(int(cu[s + 1]), out_rows)
        if b <= a:
            assert bool((out[:, s] == 0).all())
            continue
        kk = k[:, :, a:b].repeat_interleave(G, dim=1)
        vv = v[:, :, a:b].repeat_interleave(G, dim=1)
        z = (kk * q[:, s, :, None]).sum(-1) / d ** 0.5
        ref = (torch.softmax(z, -1)[..., None] * vv).sum(2)
        err = (out[:, s] - ref).abs().amax(-1) / ref.abs().amax(-1)
        assert float(err.max()) < 2.0 ** -15


@pytest.mark.parametrize("case", ["waves8", "waves16_edges_64_rows", "waves4_many_splits",
                                  "one_head_128", "few_all_heads_256", "few_all_heads_128",
                                  "all_heads", "all_heads_128_splits"])
def test_non_finite_rows_stay_in_their_sequence(case):
    """A sequence whose keys hold a NaN and infinities leaves every other sequence bit for bit as
    it was; a NaN and an infinity in V reach their own (head, dim) columns alone."""
    import torch

    from paper_2609_22158_amd import binding as B

    L, Hq, Hkv, d, rows, _ = CASES[case]
    G = Hq // Hkv
    cu = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    n = int(cu[-1])
    pb = B.Problem(L, Hq, Hkv, d, 1, cu, np.zeros(len(rows) + 1, np.int32))
    gen = torch.Generator(device="cuda").manual_seed(4)
    q = torch.randn((L, len(rows), Hq, d), generator=gen, device="cuda").to(torch.bfloat16)
    k, v = (torch.randn((L, Hkv, n, d), generator=gen, device="cuda").to(torch.bfloat16)
            for _ in range(2))
    cud = torch.from_numpy(cu).cuda()
    log(f"[decode merge non-finite {case}]")
    good = B.decode_attention(pb, q, k, v, cud, n)
    s = int(np.argmax(rows))
    a, b = int(cu[s]), int(cu[s + 1])
    bad_k = k.clone()
    bad_k[0, 0, a, 0], bad_k[0, 0, b - 1, 1] = float("inf"), float("nan")
    bad_k[0, 0, (a + b) // 2, 2] = float("-inf")
    out = B.decode_attention(pb, q, bad_k, v, cud, n)
    other = torch.ones_like(good, dtype=torch.bool)
    other[0, s, :G] = False
    assert torch.equal(out[other], good[other])
    bad_v = v.clone()
    bad_v[0, 0, a, 0], bad_v[0, 0, b - 1, 5] = float("nan"), float("inf")
    out = B.decode_attention(pb, q, k, bad_v, cud, n)
    other = torch.ones_like(good, dtype=torch.bool)
    other[0, s, :G, 0] = other[0, s, :G, 5] = False
    assert torch.equal(out[other], good[other])
    assert bool(torch.isnan(out[0, s, :G, 0]).all()) and not bool(out[0, s, :G, 5].isfinite().any())


@pytest.mark.parametrize("L,d", [(1, 64), (1, 128), (80, 64), (80, 128)])
def test_split_of_nan_alone_adds_nothing(L, d):
    """The last key, alone in its split, is NaN: the output is the attention over the other rows,
    with a few workgroups of 8 or 16 waves as with many of 4."""
    import torch

    from paper_2609_22158_amd import binding as B

    n, H, G = 1025, 2, 4
    cu = np.array([0, n], np.int32)
    gen = torch.Generator(device="cuda").manual_seed(6)
    q = torch.randn((L, 1, H * G, d), generator=gen, device="cuda").to(torch.bfloat16)
    k, v = (torch.randn((L, H, n, d), generator=gen, device="cuda").to(torch.bfloat16)
            for _ in range(2))
    k[:, :, n - 1] = float("nan")
    log(f"[decode NaN split L={L} d={d}]")
    out = []
    for rows in (n, n - 1):
        pb = B.Problem(L, H * G, H, d, 1, np.array([0, rows]), np.zeros(2, np.int32))
        out.append(B.decode_attention(pb, q, k[:, :, :rows].contiguous(), v[:, :, :rows].contiguous(),
                                      torch.from_numpy(cu).cuda().clamp(max=rows), rows))
    # the same partial states but for the merge's forms, which add in another order
    torch.testing.assert_close(out[0], out[1], rtol=1e-5, atol=1e-6)
