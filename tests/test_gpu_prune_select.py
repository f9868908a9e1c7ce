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


@pytest.mark.parametrize("kind", ["lognormal", "few", "zeros"])
@pytest.mark.parametrize("shared", [False, True], ids=["per_head", "shared"])
@pytest.mark.parametrize("lens,heads,budget,dtype", [
    ([9000, 4100, 8192, 77], 96, 8192, torch.bfloat16),   # a workgroup a row: more positions than it lists at a time
    ([4100, 900, 1, 4096], 5, 1008, torch.float32),       # several a row, the last one's share cut short or empty
    ([1000], 3, 64, torch.bfloat16), ([300, 17], 2, 512, torch.float32),   # one pass each; nothing to evict
    ([32768, 20000], 2, 16384, torch.bfloat16), ([32769, 31], 2, 4112, torch.float32),   # both sides of the two ways
    # two launches, little kept: 256 threads a chunk where the average row is longer than 32 budgets, else 512
    ([16400, 9000], 3, 256, torch.bfloat16), ([33000, 32536], 2, 1024, torch.float32), ([33000, 32538], 2, 1024, torch.bfloat16)])
def test_shares_of_the_copy(lens, heads, budget, dtype, shared, kind):
    """Every kept token of every row lands in its slot, whatever share of the row it belongs to."""
    dev, D, B = "cuda", 64, 16
    g = torch.Generator(device=dev)
    g.manual_seed(sum(lens) + budget)
    total, longest, pages = sum(lens), max(lens), budget // B
    # scores that bf16 holds; head-shared: the same in every head, so that their mean is the number itself
    score = _scores(kind, total * (1 if shared else heads), g).to(torch.bfloat16).float().view(total, -1).expand(total, heads)
    k = torch.zeros((total, heads, D), device=dev, dtype=dtype)
    v = torch.zeros_like(k)
    k[:, :, 5] = 1.0
    v[:, :, 9] = score.to(dtype)
    k[:, :, 60] = (torch.arange(total, device=dev) % 128 / 65536.0)[:, None].to(dtype)   # tells neighbours apart
    rows = () if shared else (heads,)
    table = torch.randperm(len(lens) * (1 if shared else heads) * pages, generator=g, device=dev).int().view((len(lens),) + rows + (pages,))
    shape = (table.numel(), B) + ((heads, D) if shared else (D,))
    k_pool, v_pool = torch.zeros(shape, device=dev, dtype=dtype), torch.zeros(shape, device=dev, dtype=dtype)
    out_lens = torch.zeros(len(lens), dtype=torch.int32, device=dev)
    kept = torch.full((len(lens),) + rows + (budget,), -2, dtype=torch.int32, device=dev)
    desc = pe.make_desc(dtype, len(lens), heads, heads, D, B, pages, table.numel(),
                        pe.PE_LAYOUT_SHARED if shared else pe.PE_LAYOUT_PER_HEAD)
    cu = torch.tensor([sum(lens[:i]) for i in range(len(lens) + 1)], dtype=torch.int32)
    pe.pe_prefill_prune(desc, k, v, cu.to(dev), total, longest, budget, k_pool, v_pool, table, out_lens, kept,
                        pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, total, device=dev))
    real = (v.double().square().sum(-1).sqrt() / k.double().square().sum(-1).sqrt()).float()
    if shared:
        real = real.double().mean(-1, keepdim=True).float()
    for i, n in enumerate(lens):
        keep, at = min(n, budget), torch.arange(min(n, budget), device=dev)
        assert int(out_lens[i]) == keep
        order = torch.sort(real[int(cu[i]):int(cu[i]) + n], dim=0, stable=True).indices[n - keep:]
        stay = torch.sort(order, dim=0).values.t()   # [rows, keep]
        assert torch.equal(kept[i, ..., :keep].long().view(-1, keep), stay)
        assert bool((kept[i, ..., keep:] == -1).all())
        page = table[i].long().view(-1, pages)[:, at // B]
        for pool, x in ((k_pool, k), (v_pool, v)):
            got = pool[page, at % B]   # [rows, keep, (heads,) D]
            want = x[int(cu[i]) + stay[0]][None] if shared else x[int(cu[i]) + stay, torch.arange(heads, device=dev)[:, None]]
            assert torch.equal(got, want), i
