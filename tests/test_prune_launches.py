"""A prune's selection and copy: which calls make them in one launch (the rule, on the CPU), and on the GPU that a row comes out the same
in a call that does and in one that does not."""
import os
import subprocess

import pytest
import torch

from paper_2509_04377_amd import binding as pe
from paper_2509_04377_amd import build

CHECK = r"""
#include <cstdio>
#include <cstdlib>
#include "%s/pe_place.h"
int main(int argc, char** argv) {
  printf("%%d\n", pe::prune_log2_parts(atoi(argv[1]), atoi(argv[2]), atoll(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]), 256));
}
"""


@pytest.fixture(scope="module")
def log2_parts(tmp_path_factory):
    d = tmp_path_factory.mktemp("parts")
    src, exe = d / "parts.hip", d / "parts"
    src.write_text(CHECK % build.CSRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.FLAGS + [str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)

    def run(lens, heads, budget, dim=128, elem=2, longest=None):
        args = (len(lens), heads, sum(lens), max(lens) if longest is None else longest, budget, 4 * dim * elem)
        return int(subprocess.run([str(exe)] + [str(a) for a in args], check=True, capture_output=True, text=True).stdout)
    return run


@pytest.mark.parametrize("lens,heads,budget,dim,elem,want", [
    ([4096] * 8, 8, 1024, 64, 2, 2), ([1000], 8, 1024, 128, 2, 3), ([0], 8, 64, 128, 2, 0), ([300] * 64, 8, 256, 64, 2, 0),
    # one long row among short ones, of which much is kept: its share would be copied by one compute unit while the others wait
    ([32768] + [512] * 31, 8, 16384, 128, 2, -1), ([32768] + [512] * 127, 2, 16384, 128, 2, -1), ([20000] + [300] * 63, 8, 8192, 128, 2, -1),
    ([16384] + [700] * 15, 8, 8192, 64, 4, -1), ([4096] + [128] * 16, 8, 1024, 128, 2, -1), ([4096] * 4 + [128] * 13, 8, 4096, 128, 2, -1),
    # nearly half of the compute units, or of a second round of them, without work
    ([8192] * 17, 8, 4096, 128, 2, -1), ([4096] * 33, 8, 2048, 128, 2, -1), ([9000] * 48, 8, 4096, 128, 2, -1),
    ([4096] * 32, 8, 4096, 128, 2, 0), ([16384] * 32, 8, 8192, 128, 2, 0), ([16384] * 16, 8, 8192, 128, 2, 1),
    ([17104] * 12 + [8000] * 19, 4, 3520, 128, 2, 1), ([9893] * 20 + [650] * 40, 8, 7808, 64, 2, -1),
    # half of the workgroups with a long row's share are too few
    ([16384] * 16 + [512] * 15, 8, 8192, 128, 2, -1), ([16384] * 8 + [512] * 8, 8, 8192, 128, 2, -1), ([16384] * 20 + [512] * 11, 8, 8192, 128, 2, 0),
    # up to three times what two launches copy at a time, if most compute units have a share
    ([7783] * 12 + [3927] * 12, 2, 3776, 128, 2, 2), ([4096] * 9, 8, 2048, 128, 2, 1), ([8192] * 9, 8, 4096, 128, 2, -1),
    ([16384] * 3 + [512] * 5, 8, 8192, 128, 2, -1), ([16384] * 4 + [512] * 4, 8, 8192, 128, 2, 2),
    # large shares, but no larger than what two launches copy at a time
    ([1000] * 64, 8, 1024, 128, 2, 0), ([2000] * 64, 8, 1024, 64, 2, 0), ([4096] * 4, 8, 4096, 128, 2, 3),
    # long rows of which little is kept, and what no workgroup holds
    ([30335], 2, 1120, 64, 2, -1), ([32768] * 8, 8, 1024, 128, 2, -1), ([8192], 2, 64, 64, 2, 0), ([8193], 2, 64, 64, 2, -1),
    ([9300] * 16, 8, 1024, 128, 2, 1), ([32769], 8, 8192, 128, 2, -1)])
def test_which_prunes_are_one_launch(log2_parts, lens, heads, budget, dim, elem, want):
    assert log2_parts(lens, heads, budget, dim, elem) == want


@pytest.mark.gpu
@pytest.mark.parametrize("shared", [False, True], ids=["per_head", "shared"])
@pytest.mark.parametrize("dtype,D", [(torch.bfloat16, 128), (torch.float32, 64)])
@pytest.mark.parametrize("L", [2049, 4096, 4097, 8192, 8195, 16384, 16385, 32768])
def test_one_launch_and_two(log2_parts, dtype, D, L, shared):
    """The first row of a call of one prompt, one launch, and of a call with 32 short prompts beside it, two: kept tokens and pages, bit for
    bit.  Half of the scores are equal to others, so that ties are cut too."""
    Hk, B, elem = 8, 16, dtype.itemsize
    budget = L // 2 // B * B
    g = torch.Generator(device="cuda")
    g.manual_seed(L + D)
    lens = [L] + [37] * 32
    k, v = (torch.randn((sum(lens), Hk, D), generator=g, device="cuda").to(dtype) for _ in range(2))
    k[: L // 2] = 1.0
    v[: L // 2] = torch.randint(1, 9, (L // 2, Hk, 1), generator=g, device="cuda").to(dtype) / 4
    assert log2_parts(lens, Hk, budget, D, elem) < 0 <= log2_parts(lens[:1], Hk, budget, D, elem)
    results = []
    for n in (33, 1):
        total, blocks = sum(lens[:n]), budget // B
        heads = 1 if shared else Hk
        table = torch.arange(n * heads * blocks, dtype=torch.int32, device="cuda").view((n, blocks) if shared else (n, heads, blocks))
        pool = (n * heads * blocks, B, Hk, D) if shared else (n * heads * blocks, B, D)
        k_pool, v_pool = torch.zeros(pool, dtype=dtype, device="cuda"), torch.zeros(pool, dtype=dtype, device="cuda")
        desc = pe.make_desc(dtype, n, Hk, Hk, D, B, blocks, pool[0], pe.PE_LAYOUT_SHARED if shared else pe.PE_LAYOUT_PER_HEAD)
        cu = torch.tensor([0] + lens[:n], device="cuda").cumsum(0).int()
        out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        kept = torch.full((n, heads, budget), -7, dtype=torch.int32, device="cuda")
        pe.pe_prefill_prune(desc, k[:total], v[:total], cu, total, L, budget, k_pool, v_pool, table, out, kept,
                            pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, total, device="cuda"))
        assert out.tolist() == [min(x, budget) for x in lens[:n]]
        if n > 1:   # the short ones are kept whole
            assert torch.equal(kept[1:, :, :37], torch.arange(37, device="cuda").int().expand(n - 1, heads, 37))
            assert bool((kept[1:, :, 37:] == -1).all())
        results.append((kept[0], k_pool[: heads * blocks].view(torch.uint8), v_pool[: heads * blocks].view(torch.uint8)))
    assert bool((results[0][0][:, 1:] > results[0][0][:, :-1]).all()) and int(results[0][0].min()) >= 0
    for a, b in zip(*results):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("L,said", [(1010, 1000), (1024, 513), (4000, 3073)])
def test_a_row_somewhat_longer_than_said(log2_parts, L, said):
    """A bound on the lengths that is too small by less than 1024 tokens, as it was taken by launches for whole chunks of them: the same
    result as with the right one."""
    Hk, B, D, budget = 4, 16, 64, 512
    assert log2_parts([L], Hk, budget, D, 2, said) >= 0
    g = torch.Generator(device="cuda")
    g.manual_seed(L)
    k, v = (torch.randn((L, Hk, D), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    blocks = budget // B
    table = torch.arange(Hk * blocks, dtype=torch.int32, device="cuda").view(1, Hk, blocks)
    desc = pe.make_desc(torch.bfloat16, 1, Hk, Hk, D, B, blocks, Hk * blocks)
    cu = torch.tensor([0, L], dtype=torch.int32, device="cuda")
    results = []
    for longest in (L, said):
        pools = [torch.zeros((Hk * blocks, B, D), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        out = torch.zeros(1, dtype=torch.int32, device="cuda")
        kept = torch.full((1, Hk, budget), -7, dtype=torch.int32, device="cuda")
        pe.pe_prefill_prune(desc, k, v, cu, L, longest, budget, *pools, table, out, kept,
                            pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, L, device="cuda"))
        results.append(pools + [out, kept])
    assert int(results[0][3].min()) >= 0
    for a, b in zip(*results):
        assert torch.equal(a, b)
