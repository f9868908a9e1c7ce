"""The merge of a row's splits at the counts where it changes from one wave to four and to eight, against the whole row."""
import pytest
import torch

from paper_2509_04377_amd import binding as pe

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("splits", [2, 8, 9, 12, 32, 33, 64, 131, 256])
@pytest.mark.parametrize("dtype,D,G,Hk,n", [(torch.float32, 64, 3, 2, 3001), (torch.float32, 128, 1, 8, 517), (torch.bfloat16, 64, 8, 1, 9000),
                                            (torch.bfloat16, 128, 4, 8, 2100), (torch.bfloat16, 64, 1, 3, 40),
                                            (torch.bfloat16, 128, 8, 8, 2500)])   # (in twelve: eight waves by one, and a merge launch)
def test_merge_of_many_splits(dtype, D, G, Hk, n, splits):
    """Either side adds the same products in its own order: at most n + splits roundings to fp32, of sums that are no larger than the
    largest value, but what is rounded at random adds up as the root of their number (eight times that is allowed); for bf16 one
    rounding of the output on either side."""
    B, S = 16, 2
    g = torch.Generator(device=DEV)
    g.manual_seed(n + splits)
    lens = [n, max(1, n // 3)]
    pages = -(-n // B)
    table = torch.randperm(S * Hk * pages, generator=g, device=DEV).int().view(S, Hk, pages)
    k, v = (torch.randn((S * Hk * pages, B, D), generator=g, device=DEV).to(dtype) for _ in range(2))
    q = torch.randn((S, G * Hk, D), generator=g, device=DEV).to(dtype)
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    outs = []
    for count in (1, splits):
        desc = pe.make_desc(dtype, S, Hk, G * Hk, D, B, pages, S * Hk * pages, decode_splits=count)
        out = torch.full_like(q, 9.0)
        pe.pe_paged_decode(desc, q, k, v, table, sl, D ** -0.5, out, pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc, device=DEV))
        outs.append(out.double())
    tol = 8 * (n + splits) ** 0.5 * 2.0 ** -24 * float(v.abs().max())
    if dtype == torch.bfloat16:
        tol = tol + 2.0 ** -7 * outs[0].abs()
    assert bool(((outs[0] - outs[1]).abs() <= tol).all()), float((outs[0] - outs[1]).abs().max())
