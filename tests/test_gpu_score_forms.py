"""The block scores of a large table, whose sweep takes two or four pages a wave, against the same rows scored in slices, whose sweeps take
one (and are compared with the oracle elsewhere): bit for bit, in every mode."""
import pytest
import torch

from paper_2509_04377_amd import binding as pe

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("shared", [False, True], ids=["per_head", "shared"])
@pytest.mark.parametrize("dtype,D,B,seqs,max_blocks", [
    (torch.bfloat16, 64, 16, 512, 16), (torch.bfloat16, 64, 16, 2048, 19),       # two pages a wave, four
    (torch.float32, 64, 16, 512, 15), (torch.bfloat16, 128, 32, 1024, 9), (torch.float32, 128, 32, 2048, 17),
    (torch.bfloat16, 64, 64, 1024, 9), (torch.float32, 64, 128, 2048, 33), (torch.bfloat16, 128, 128, 4096, 5)])
def test_pages_a_wave(dtype, D, B, seqs, max_blocks, shared):
    Hk, P = 8, 300
    g = torch.Generator(device=DEV)
    g.manual_seed(seqs + max_blocks)
    shape = (P, B, Hk, D) if shared else (P, B, D)
    k, v = (torch.randn(shape, generator=g, device=DEV).to(dtype) for _ in range(2))
    # (the calls only read the pages: rows may share them here)
    table = torch.randint(0, P, (seqs, max_blocks) if shared else (seqs, Hk, max_blocks), generator=g, device=DEV, dtype=torch.int32)
    budget = max(1, max_blocks // 2) * B
    lens = torch.randint(0, max_blocks * B + 1, (seqs,), generator=g, device=DEV, dtype=torch.int32)
    lens[::3] = lens[::3] // B * B   # some that trigger
    layout = pe.PE_LAYOUT_SHARED if shared else pe.PE_LAYOUT_PER_HEAD

    def run(part, mode):
        n = len(range(*part.indices(seqs)))
        desc = pe.make_desc(dtype, n, Hk, Hk, D, B, max_blocks, P, layout)
        scores = torch.full((n, Hk, max_blocks), -1.0, device=DEV)
        t, ln = table[part].contiguous(), lens[part].contiguous()
        if mode == "all":
            pe.pe_score_blocks(desc, k, v, t, ln, scores)
        elif mode == "triggered":
            pe.pe_score_triggered_blocks(desc, k, v, t, ln, budget, scores)
        else:
            pe.pe_score_recent_blocks(desc, k, v, t, ln, mode, scores)
        return scores

    for mode in ("all", "triggered", 1, max_blocks - 1):
        whole = run(slice(0, seqs), mode)
        for at in range(0, seqs, 64):
            part = slice(at, min(seqs, at + 64))
            assert torch.equal(whole[part].view(torch.int32), run(part, mode).view(torch.int32)), (mode, at)
