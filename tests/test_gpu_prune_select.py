"""The selection of the prefill prune against a stable sort, over score distributions that take each of its ways: few candidates,
several digits, more candidates than LDS holds, equal scores, zeros and infinities, and rows at the edges of what a workgroup holds."""
import pytest
import torch

from paper_2509_04377_amd import binding as pe

pytestmark = pytest.mark.gpu

HOLDINGS = [[1, 3, 255, 257, 1023, 4095, 4096], [4097, 2, 8191, 8192], [16383, 16384, 1025, 8193], [16385, 6, 32767, 32768, 1024],
            [32769, 40001, 65535, 65536, 100], [65537, 70001, 5, 131075],
            [40000, 1, 4095, 4097, 8192, 12289, 61440, 61441, 300]]


def _scores(kind, n, g):
    """Non-negative fp32 scores."""
    dev = g.device
    z = torch.randn(n, generator=g, device=dev)
    if kind == "lognormal":
        return torch.exp(0.7 * z)
    if kind == "wide":        # more than the exponent range of a histogram of narrow bins
        return torch.exp(12 * z)
    if kind == "equal":
        return torch.full((n,), 1.25, device=dev)
    if kind == "few":         # some hundred distinct values: every bin holds many equal ones
        return torch.exp(0.7 * z).mul(16).round().clamp(min=1) / 16
    if kind == "neighbours":  # consecutive fp32 numbers, all in a few bins of any histogram over the row's range and an outlier
        bits = torch.randint(0, 5000, (n,), generator=g, device=dev, dtype=torch.int32) + 0x3f800000
        s = bits.view(torch.float32).clone()
        s[n // 2] = 1e30
        return s
    if kind in ("zeros", "infinities"):   # so many that the threshold is one of them for some of the budgets
        s = torch.exp(0.7 * z)
        s[torch.rand(n, generator=g, device=dev) < 0.6] = 0.0 if kind == "zeros" else float("inf")
        return s
    if kind == "neither":     # nothing else: no sample to lay a histogram over
        return torch.where(torch.rand(n, generator=g, device=dev) < 0.5, 0.0, float("inf"))
    s = torch.exp(0.7 * z)    # "edges": zeros and infinities among them
    s[::37] = 0.0
    s[5::41] = float("inf")
    return s


@pytest.mark.parametrize("lens", HOLDINGS, ids=lambda v: str(max(v)))
@pytest.mark.parametrize("kind", ["lognormal", "wide", "equal", "few", "neighbours", "edges", "zeros", "infinities",
                                  "neither"])
def test_selection_is_a_stable_sort(lens, kind):
    dev, D, B, Hk = "cuda", 64, 16, 2
    g = torch.Generator(device=dev)
    g.manual_seed(len(kind) * 1000 + max(lens))
    total, longest = sum(lens), max(lens)
    # one element per row: the score is |V| / |K| = the number itself (0 for V = 0, infinity for K = 0)
    score = torch.stack([_scores(kind, total, g) for _ in range(Hk)], 1)
    k = torch.zeros((total, Hk, D), device=dev)
    v = torch.zeros_like(k)
    k[:, :, 3] = torch.where(torch.isinf(score), 0.0, 1.0)
    v[:, :, 7] = torch.where(torch.isinf(score), 1.0, score)
    cu = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32)
    for budget in (16, 1024 if longest > 1024 else 512, (longest - 1) // B * B):
        pages = -(-budget // B)
        table = torch.arange(len(lens) * Hk * pages, dtype=torch.int32, device=dev).view(len(lens), Hk, pages)
        pool = torch.zeros((table.numel(), B, D), device=dev)
        v_pool, out_lens = torch.zeros_like(pool), torch.zeros(len(lens), dtype=torch.int32, device=dev)
        kept = torch.full((len(lens), Hk, budget), -2, dtype=torch.int32, device=dev)
        desc = pe.make_desc(torch.float32, len(lens), Hk, Hk, D, B, pages, table.numel())
        ws = pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, total, device=dev)
        pe.pe_prefill_prune(desc, k, v, cu.to(dev), total, longest, budget, pool, v_pool, table, out_lens, kept, ws)
        for i, n in enumerate(lens):
            keep = min(n, budget)
            assert int(out_lens[i]) == keep
            for h in range(Hk):
                row = score[int(cu[i]):int(cu[i]) + n, h]
                stay = torch.sort(torch.sort(row, stable=True).indices[n - keep:]).values
                assert torch.equal(kept[i, h, :keep].long(), stay), (budget, i, h)
                assert bool((kept[i, h, keep:] == -1).all())
                at = torch.arange(keep, device=dev)
                got = v_pool[table[i, h].long()[at // B], at % B, 7]
                assert torch.equal(got, v[int(cu[i]) + stay, h, 7]), (budget, i, h)
