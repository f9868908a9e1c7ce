"""Which (row, split) an attention workgroup owns: the division-free grid against the plain division, on the CPU, and the grids
that are divided (more rows than a grid has) on the GPU."""
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
  const int S = atoi(argv[1]), H = atoi(argv[2]), n = atoi(argv[3]), step = atoi(argv[4]);
  for (int xcd = 0; xcd < 2; ++xcd) {
    pe::PlaceGrid g;
    if (!pe::place_grid(S, H, n, xcd != 0, &g)) return 2;
    const int64_t rows = (int64_t)S * H;
    if ((int64_t)g.x * g.y != rows * n || g.xcd != (xcd && rows %% 8 == 0)) return 3;
    if (g.y > 65535) return 4;
    for (int64_t b = 0; b < rows * n; b += b + step < rows * n || b == rows * n - 1 ? step : rows * n - 1 - b) {
      const pe::Place p = pe::place_at((uint32_t)(b %% g.x), (uint32_t)(b / g.x), g.xcd, g.linear, n, H, g.inv_heads);
      const int64_t row = g.xcd ? b / 8 / n * 8 + b %% 8 : b / n, split = g.xcd ? b / 8 %% n : b %% n;
      if (p.row != row || p.split != split || p.seq != row / H || p.head != row %% H) {
        printf("workgroup %%lld: row %%d split %%d seq %%d head %%d\n", (long long)b, p.row, p.split, p.seq, p.head);
        return 1;
      }
    }
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    d = tmp_path_factory.mktemp("place")
    src, exe = d / "place.hip", d / "place"
    src.write_text(CHECK % build.CSRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.FLAGS + [str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)
    return str(exe)


@pytest.mark.parametrize("S,H,splits", [(1, 1, 1), (1, 1, 256), (3, 7, 5), (8, 3, 4), (32, 8, 1), (48, 8, 64), (1, 130, 2), (65535, 1, 1),
                                        (65536, 1, 1), (65535, 8, 2), (65536, 8, 2), (21845, 24, 1), (40000, 13, 3),
                                        (7, 65537, 2), (1, 1 << 20, 1), (3, 1 << 23, 4)])
def test_place_is_the_division(checker, S, H, splits):
    step = max(1, S * H * splits // 1000003)
    assert subprocess.run([checker, str(S), str(H), str(splits), str(step)]).returncode == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("S,Hk,splits", [(70001, 1, 1), (35003, 2, 2), (65544, 8, 1), (9, 7, 3), (8, 3, 5)])
def test_attention_over_many_rows(dt, S, Hk, splits):
    """Rows beyond a grid's 65535 (with and without the order by XCD), and odd counts of rows and heads."""
    dev, B, D, pages, G = "cuda", 16, 64, 2, 1 if S > 1000 else 3
    dtype = torch.float32 if dt == "f32" else torch.bfloat16
    g = torch.Generator(device=dev)
    g.manual_seed(S + splits)
    P = 257
    k, v = (torch.randn((P, B, D), generator=g, device=dev).to(dtype) for _ in range(2))
    table = torch.randint(0, P, (S, Hk, pages), generator=g, device=dev, dtype=torch.int32)   # only read here: rows may share pages
    lens = torch.randint(1, pages * B + 1, (S,), generator=g, device=dev, dtype=torch.int32)
    q = torch.randn((S, Hk * G, D), generator=g, device=dev).to(dtype)
    desc = pe.make_desc(dtype, S, Hk, Hk * G, D, B, pages, P, decode_splits=splits)
    out = torch.empty_like(q)
    pe.pe_paged_decode(desc, q, k, v, table, lens, D ** -0.5, out, pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc, device=dev))
    step = max(1, 16384 // Hk)
    tol = 1e-5 if dt == "f32" else 2e-2
    for s0 in range(0, S, step):
        t = table[s0:s0 + step].long()
        kk, vv = (x[t].float().flatten(2, 3) for x in (k, v))                       # [s, Hk, pages * B, D]
        qq = q[s0:s0 + step].float().view(t.shape[0], Hk, G, 1, D)
        logits = (qq * kk[:, :, None]).sum(-1) * D ** -0.5
        dead = torch.arange(pages * B, device=dev)[None, :] >= lens[s0:s0 + step, None]
        p = torch.softmax(logits.masked_fill(dead[:, None, None, :], float("-inf")), -1)
        want = (p[..., None] * vv[:, :, None]).sum(-2)
        got = out[s0:s0 + step].float().view(want.shape)
        err = (got - want).norm(dim=-1) / want.norm(dim=-1)
        assert float(err.max()) <= tol, (s0, float(err.max()))


PIECES = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "%s/pe_place.h"
int main(int argc, char** argv) {
  const int S = atoi(argv[1]), rows = atoi(argv[2]), chunks = atoi(argv[3]), threads = 256;
  std::vector<int64_t> next(1, 0);   // pairs come in whole rectangles, sequences slowest
  int64_t covered = 0, launches = 0, s_at = 0, c_at = 0;
  const bool all = pe::launch_pieces(S, rows, chunks, threads, [&](int s0, int ns, int c0, int nc) {
    if (ns < 1 || nc < 1 || (int64_t)ns * rows * nc * threads >= (1LL << 32)) exit(2);
    if (s0 != s_at || c0 != c_at || s0 + ns > S || c0 + nc > chunks) exit(3);
    c_at += nc;
    if (c_at == chunks) c_at = 0, s_at += ns;
    covered += (int64_t)ns * nc;
    return ++launches < 1000000;
  });
  if (all != (rows < (1 << 24))) return 4;
  if (all && (covered != (int64_t)S * chunks || s_at != S)) return 5;
  printf("%%lld\n", (long long)launches);
  return 0;
}
"""


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    src, exe = d / "pieces.hip", d / "pieces"
    src.write_text(PIECES % build.CSRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.FLAGS + [str(src), "-o", str(exe)], check=True, stderr=subprocess.DEVNULL)
    return str(exe)


@pytest.mark.parametrize("S,rows,chunks,launches", [
    (1, 1, 1, 1), (32, 8, 16, 1), (4096, 8, 511, 1), (4096, 8, 512, 2), (4095, 8, 512, 1), (65536, 8, 100, 4), (1 << 21, 8, 1, 2),
    (4194303, 7, 3, 6), (3, (1 << 24) - 1, 2, 6), (1, 1 << 24, 1, 0), (1, 5, 1 << 21, 1), (1, 1, (1 << 24) - 1, 1), (1, 1, 1 << 24, 2)])
def test_launch_pieces_cover_every_pair_once(pieces, S, rows, chunks, launches):
    r = subprocess.run([pieces, str(S), str(rows), str(chunks)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and int(r.stdout) == launches


@pytest.mark.gpu
def test_head_shared_prune_of_many_head_chunk_pairs():
    """2^24 (head, chunk) pairs, more than one launch takes: the bound on the lengths sizes the launch, not the lengths."""
    dev, S, Hk, D, B, n = "cuda", 4096, 8, 64, 16, 128
    total = S * n
    k, v = (torch.zeros((total, Hk, D), dtype=torch.bfloat16, device=dev) for _ in range(2))
    g = torch.Generator(device=dev)
    g.manual_seed(11)
    k[:, :, 0] = 1.0
    score = torch.rand((S, n), generator=g, device=dev).argsort(-1).float() + 1.0    # 1 .. 128, exact in bfloat16
    v[:, :, 1] = score.view(-1, 1).to(torch.bfloat16)
    v[:, :, 2] = torch.arange(Hk, device=dev) / 1024.0   # too small to change the order; tells the heads apart
    table = torch.randperm(S, generator=g, device=dev).int().view(S, 1)
    k_pool, v_pool = (torch.zeros((S, B, Hk, D), dtype=torch.bfloat16, device=dev) for _ in range(2))
    lens, kept = torch.zeros(S, dtype=torch.int32, device=dev), torch.zeros((S, B), dtype=torch.int32, device=dev)
    desc = pe.make_desc(torch.bfloat16, S, Hk, Hk, D, B, 1, S, pe.PE_LAYOUT_SHARED)
    cu = torch.arange(S + 1, dtype=torch.int32, device=dev) * n
    ws = pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, total, device=dev)
    pe.pe_prefill_prune(desc, k, v, cu, total, total, B, k_pool, v_pool, table, lens, kept, ws)
    stay = score.topk(B, -1).indices.sort(-1).values
    assert bool((lens == B).all()) and torch.equal(kept.long(), stay)
    src = (stay + torch.arange(S, device=dev)[:, None] * n).view(-1)
    assert torch.equal(v_pool[table[:, 0].long()].view(S * B, Hk, D), v[src])
    assert torch.equal(k_pool[table[:, 0].long()].view(S * B, Hk, D), k[src])
