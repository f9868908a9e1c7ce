"""GPU parity: each C-ABI call against the CPU oracle on the same seeded inputs, element by element.

Bars: tables, lengths, eviction decisions, kept indices and pruned pool contents bit-exact; scores equal
as fp32 up to one unit in the last place (both sides compute in fp64 and round once; only the order of
fp64 additions differs); attention within 1e-5 (fp32) / 2e-2 (bf16) relative, per output vector, in the
2-norm and in the max-norm.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_04377_amd import binding as pe

from _util import f32, i32, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
TOL = {"f32": 1e-5, "bf16": 2e-2}


def _ulp_diff(a: np.ndarray, b: np.ndarray) -> np.ndarray:
    """Distance in fp32 representable steps (inputs are non-negative floats or +inf)."""
    return np.abs(a.view(np.int32).astype(np.int64) - b.view(np.int32).astype(np.int64))


def make_paged(seed, lens, Hk, D, B, dtype, extra=1, pad_pages=3):
    """Random rows in shuffled pages (torch CPU tensors in `dtype`); unused slots hold junk."""
    g = torch.Generator().manual_seed(seed)
    S = len(lens)
    nb = [(L + B - 1) // B for L in lens]
    mb = max(max(nb), 1) + extra
    P = Hk * sum(nb) + pad_pages
    ids = torch.randperm(P, generator=g).to(torch.int32)
    table = torch.full((S, Hk, mb), -1, dtype=torch.int32)
    pos = 0
    for s in range(S):
        for h in range(Hk):
            table[s, h, :nb[s]] = ids[pos:pos + nb[s]]
            pos += nb[s]
    sc_k = torch.exp(0.5 * torch.randn((P, B, 1), generator=g))
    sc_v = torch.exp(0.5 * torch.randn((P, B, 1), generator=g))
    k_pool = (torch.randn((P, B, D), generator=g) * sc_k).to(dtype)
    v_pool = (torch.randn((P, B, D), generator=g) * sc_v).to(dtype)
    return k_pool, v_pool, table, torch.tensor(lens, dtype=torch.int32)


def gpu_scores(k_pool, v_pool, table, lens, Hq=None):
    P, B, D = k_pool.shape
    S, Hk, mb = table.shape
    desc = pe.make_desc(k_pool.dtype, S, Hk, Hq or Hk, D, B, mb, P)
    out = torch.full((S, Hk, mb), -123.0, dtype=torch.float32, device=DEV)
    pe.pe_score_blocks(desc, k_pool.to(DEV), v_pool.to(DEV), table.to(DEV), lens.to(DEV), out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B", [16, 32, 64, 128])
def test_score_blocks_random(dt, D, B):
    print("case score_blocks_random", dt, D, B, flush=True)
    # 37 pages per row at most: three 16-page groups with a ragged tail; a partial tail page; an empty row
    lens = [37 * B, 20 * B + 5, 0, B, 16 * B]
    k_pool, v_pool, table, sl = make_paged(100 + D + B, lens, 3, D, B, DTYPES[dt], extra=2)
    got = gpu_scores(k_pool, v_pool, table, sl)
    want = oracle.score_blocks(f32(k_pool), f32(v_pool), i32(table), i32(sl))
    assert np.array_equal(np.isinf(got), np.isinf(want))
    fin = np.isfinite(want)
    ulp = _ulp_diff(got[fin], want[fin])
    assert ulp.max() <= 1, "score differs by more than one fp32 step"
    assert (ulp != 0).mean() < 1e-3, "scores should be bit-equal except at rare rounding boundaries"


def test_score_triggered_blocks_touches_only_sequences_that_evict():
    print("case score_triggered_blocks", flush=True)
    B, D, Hk = 16, 128, 3
    C = 4 * B
    lens = [8 * B, 8 * B - 1, 3 * B, 0, 4 * B, 9 * B + 5, 20 * B]   # triggers: 0, 4, 6 (3*B is under budget)
    k_pool, v_pool, table, sl = make_paged(150, lens, Hk, D, B, torch.bfloat16, extra=2)
    S, _, mb = table.shape
    desc = pe.make_desc(torch.bfloat16, S, Hk, Hk, D, B, mb, k_pool.shape[0])
    got = torch.full((S, Hk, mb), -123.0, dtype=torch.float32, device=DEV)
    pe.pe_score_triggered_blocks(desc, k_pool.to(DEV), v_pool.to(DEV), table.to(DEV), sl.to(DEV), C, got)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    want = oracle.score_blocks(f32(k_pool), f32(v_pool), i32(table), i32(sl))
    for s, L in enumerate(lens):
        if L > 0 and L % B == 0 and L >= C:
            assert np.array_equal(got[s].view(np.int32), want[s].view(np.int32)), s   # bf16: sums are exact
        else:
            assert np.all(got[s] == np.float32(-123.0)), s
    assert [s for s in range(S) if got[s, 0, 0] != np.float32(-123.0)] == [0, 4, 6]


def test_score_blocks_closed_forms():
    print("case score_blocks_closed_forms", flush=True)
    B, D, Hk = 16, 128, 2
    lens = [8 * B]
    k_pool, v_pool, table, sl = make_paged(7, lens, Hk, D, B, torch.bfloat16)
    # V = K  ->  exactly 1
    got = gpu_scores(k_pool, k_pool.clone(), table, sl)
    assert np.all(got[:, :, :8] == np.float32(1.0)) and np.all(np.isinf(got[:, :, 8:]))
    # one-hot dyadic rows -> exact dyadic means; zero V row -> 0; zero K row -> +inf page
    g = torch.Generator().manual_seed(8)
    P = k_pool.shape[0]
    ek = torch.randint(-3, 4, (P, B), generator=g)
    ev = torch.randint(-3, 4, (P, B), generator=g)
    k1 = torch.zeros((P, B, D)); v1 = torch.zeros((P, B, D))
    col_k = torch.randint(0, D, (P, B), generator=g); col_v = torch.randint(0, D, (P, B), generator=g)
    k1.scatter_(2, col_k[..., None], (2.0 ** ek)[..., None].float())
    v1.scatter_(2, col_v[..., None], (2.0 ** ev)[..., None].float())
    zero_v_page, zero_k_page = int(table[0, 0, 1]), int(table[0, 1, 2])
    v1[zero_v_page, 3] = 0
    k1[zero_k_page, 9] = 0
    got = gpu_scores(k1.to(torch.bfloat16), v1.to(torch.bfloat16), table, sl)
    want = oracle.score_blocks(k1.numpy(), v1.numpy(), i32(table), i32(sl))
    assert np.array_equal(got.view(np.int32), want.view(np.int32))
    ratio = (2.0 ** (ev - ek).double())
    ratio[zero_v_page, 3] = 0
    exact = ratio[int(table[0, 0, 1])].sum().item() / B
    assert got[0, 0, 1] == np.float32(exact) and np.isinf(got[0, 1, 2])


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B", [16, 32, 64, 128])
@pytest.mark.parametrize("want_scores", [True, False])
def test_score_evict_one_pass(dt, D, B, want_scores):
    """pe_score_evict against oracle score_blocks + evict_blocks: odd and even page counts, one page, a partial
    tail (no trigger), under budget (no trigger), an empty row, more rows than waves (Hk = 5)."""
    print("case score_evict", dt, D, B, want_scores, flush=True)
    Hk, C = 5, 2 * B
    lens = [37 * B, 20 * B + 5, 0, B, 16 * B, 2 * B, 3 * B, 65 * B]
    k_pool, v_pool, table, sl = make_paged(900 + D + B, lens, Hk, D, B, DTYPES[dt], extra=2)
    S, _, mb = table.shape
    P = k_pool.shape[0]
    desc = pe.make_desc(k_pool.dtype, S, Hk, Hk, D, B, mb, P)
    t_gpu, l_gpu = table.to(DEV), sl.to(DEV)
    sc_gpu = torch.full((S, Hk, mb), -123.0, dtype=torch.float32, device=DEV)
    ev_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    fr_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    kd, vd = k_pool.to(DEV), v_pool.to(DEV)
    o_table, o_lens = i32(table).copy(), i32(sl).copy()
    for call in range(2):   # the second call sees the shrunken rows: only rows still at budget go again
        trig = [(L > 0 and L % B == 0 and L >= C) for L in o_lens]
        want_sc = oracle.score_blocks(f32(k_pool), f32(v_pool), o_table, o_lens)
        pe.pe_score_evict(desc, kd, vd, t_gpu, l_gpu, C, sc_gpu if want_scores else None, ev_gpu, fr_gpu)
        torch.cuda.synchronize()
        if want_scores:
            got_sc = sc_gpu.cpu().numpy()
            for s in range(S):
                if not trig[s]:
                    assert np.all(got_sc[s] == np.float32(-123.0)), "rows of idle sequences stay untouched"
                    continue
                assert np.array_equal(np.isinf(got_sc[s]), np.isinf(want_sc[s]))
                fin = np.isfinite(want_sc[s])
                assert _ulp_diff(got_sc[s][fin], want_sc[s][fin]).max() <= 1
            # the decision, taken on the scores the kernel itself reports
            dec_sc = np.where(np.array(trig)[:, None, None], got_sc, want_sc).astype(np.float32)
            t2, l2 = o_table.copy(), o_lens.copy()
            ev2, fr2 = oracle.evict_blocks(dec_sc, t2, l2, B, C)
            assert np.array_equal(ev_gpu.cpu().numpy(), ev2) and np.array_equal(fr_gpu.cpu().numpy(), fr2)
        ev, fr = oracle.evict_blocks(want_sc, o_table, o_lens, B, C)
        assert np.array_equal(ev_gpu.cpu().numpy(), ev), call
        assert np.array_equal(fr_gpu.cpu().numpy(), fr), call
        assert np.array_equal(t_gpu.cpu().numpy(), o_table), call
        assert np.array_equal(l_gpu.cpu().numpy(), o_lens), call
        assert sum(trig) == (5 if call == 0 else 4)
        sc_gpu.fill_(-123.0)


def test_score_evict_ties_and_planted_minimum():
    """All pages equal (V = K, score exactly 1) -> page 0 goes; a planted low page at the end of an odd row, at
    the end of an even row and in the middle -> exactly that page goes."""
    print("case score_evict ties", flush=True)
    B, D, Hk = 16, 128, 2
    lens = [9 * B, 10 * B, 33 * B]
    k_pool, _, table, sl = make_paged(77, lens, Hk, D, B, torch.bfloat16)
    v_pool = k_pool.clone()
    plant = {(0, 0): 8, (1, 1): 9, (2, 0): 17}   # (sequence, head) -> logical page with V halved
    for (s, h), j in plant.items():
        v_pool[int(table[s, h, j])] *= 0.5
    S, _, mb = table.shape
    desc = pe.make_desc(k_pool.dtype, S, Hk, Hk, D, B, mb, k_pool.shape[0])
    t_gpu, l_gpu = table.to(DEV), sl.to(DEV)
    ev_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    fr_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    pe.pe_score_evict(desc, k_pool.to(DEV), v_pool.to(DEV), t_gpu, l_gpu, 2 * B, None, ev_gpu, fr_gpu)
    torch.cuda.synchronize()
    ev = ev_gpu.cpu().numpy()
    for s in range(S):
        for h in range(Hk):
            j = plant.get((s, h), 0)
            assert ev[s, h] == j
            assert fr_gpu[s, h].item() == int(table[s, h, j])
    assert l_gpu.cpu().tolist() == [L - B for L in lens]


def test_evict_blocks_bit_exact():
    print("case evict_blocks_bit_exact", flush=True)
    rng = np.random.default_rng(300)
    B, Hk = 16, 5
    n_pages = [1, 2, 63, 64, 65, 128, 129, 300, 7, 40, 256, 0]
    S = len(n_pages)
    mb = 301
    lens = np.array([n * B for n in n_pages], np.int32)
    lens[8] -= 3            # tail not full -> no trigger
    C = 2 * B               # sequence 0 (one page) is under budget
    scores = rng.integers(0, 6, size=(S, Hk, mb)).astype(np.float32) * 0.25   # many exact ties
    scores[5, 0, :] = 1.0                                                      # all-tie row -> page 0
    scores[7, 1, 299] = -1.0                                                   # winner is the last page
    scores[7, 2, 64] = -1.0                                                    # winner at a pass boundary
    table = np.full((S, Hk, mb), -1, np.int32)
    ids = rng.permutation(S * Hk * mb).astype(np.int32)
    pos = 0
    for s in range(S):
        n = (lens[s] + B - 1) // B
        for h in range(Hk):
            table[s, h, :n] = ids[pos:pos + n]
            pos += n
    desc = pe.make_desc(torch.float32, S, Hk, Hk, 64, B, mb, S * Hk * mb)
    t_gpu = torch.tensor(table, device=DEV)
    l_gpu = torch.tensor(lens, device=DEV)
    ev_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    fr_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    for call in range(3):   # three rounds: rows keep shrinking, winners move
        ev, fr = oracle.evict_blocks(scores, table, lens, B, C)
        pe.pe_evict_blocks(desc, torch.tensor(scores, device=DEV), t_gpu, l_gpu, C, ev_gpu, fr_gpu)
        torch.cuda.synchronize()
        assert np.array_equal(ev_gpu.cpu().numpy(), ev), call
        assert np.array_equal(fr_gpu.cpu().numpy(), fr), call
        assert np.array_equal(t_gpu.cpu().numpy(), table), call
        assert np.array_equal(l_gpu.cpu().numpy(), lens), call
    assert (ev >= 0).any() and (ev < 0).any()


def test_evict_blocks_nan_scores_stay_inside_the_row():
    """Scores that are all NaN (finite K/V never produce one) must not send the compaction outside the table row:
    the first candidate page goes.  A NaN among real scores never wins."""
    print("case evict_blocks_nan", flush=True)
    B, Hk, S, mb = 16, 3, 4, 70
    n_pages = [5, 66, 8, 12]
    lens = np.array([n * B for n in n_pages], np.int32)
    rng = np.random.default_rng(310)
    table = np.full((S, Hk, mb), -1, np.int32)
    for s in range(S):
        for h in range(Hk):
            table[s, h, :n_pages[s]] = rng.permutation(1000)[:n_pages[s]] + 1000 * (s * Hk + h)
    scores = np.full((S, Hk, mb), np.nan, np.float32)
    scores[2, 1, :8] = [3, np.nan, 2, 2, np.nan, 5, 9, 4]       # a NaN among real scores: first minimum is page 2
    desc = pe.make_desc(torch.float32, S, Hk, Hk, 64, B, mb, 1000 * S * Hk)
    for opts, lo in ((None, 0), (dict(protect_first=3), 3), (dict(share_heads=1), 0),
                     (dict(share_heads=1, protect_first=2, protect_last=1), 2)):
        t_gpu, l_gpu = torch.tensor(table, device=DEV), torch.tensor(lens, device=DEV)
        ev_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
        fr_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
        if opts is None:
            pe.pe_evict_blocks(desc, torch.tensor(scores, device=DEV), t_gpu, l_gpu, 2 * B, ev_gpu, fr_gpu)
        else:
            o = pe.pe_evict_opts(0, opts.get("protect_first", 0), opts.get("protect_last", 0), opts.get("share_heads", 0), 0)
            pe.pe_evict_blocks_ex(desc, o, torch.tensor(scores, device=DEV), t_gpu, l_gpu, 2 * B, ev_gpu, fr_gpu)
        torch.cuda.synchronize()
        ev, fr, t_new = ev_gpu.cpu().numpy(), fr_gpu.cpu().numpy(), t_gpu.cpu().numpy()
        for s in range(S):
            for h in range(Hk):
                want = lo
                if opts is None and (s, h) == (2, 1):
                    want = 2
                assert ev[s, h] == want, (opts, s, h, ev[s, h])
                assert fr[s, h] == table[s, h, want]
                assert np.array_equal(t_new[s, h, :n_pages[s] - 1], np.delete(table[s, h, :n_pages[s]], want))
                assert np.all(t_new[s, h, n_pages[s] - 1:] == -1)
        assert np.array_equal(l_gpu.cpu().numpy(), lens - B)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("D,B", [(64, 16), (128, 16), (64, 32), (128, 32), (128, 64), (64, 128)])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 6, 8])
def test_paged_decode_shapes(dt, D, B, G):
    print("case paged_decode_shapes", dt, D, B, G, flush=True)
    Hk = 2
    lens = [0, 1, 15, 16, 17, 100, 700, 1300]
    k_pool, v_pool, table, sl = make_paged(400 + D + B + G, lens, Hk, D, B, DTYPES[dt])
    g = torch.Generator().manual_seed(401)
    S, Hq = len(lens), Hk * G
    q = torch.randn((S, Hq, D), generator=g).to(DTYPES[dt])
    want = oracle.paged_decode(f32(q), f32(k_pool), f32(v_pool), i32(table), i32(sl))
    P, mb = k_pool.shape[0], table.shape[2]
    desc = pe.make_desc(DTYPES[dt], S, Hk, Hq, D, B, mb, P)
    kd, vd, td, ld, qd = (x.to(DEV) for x in (k_pool, v_pool, table, sl, q))
    try:
        for splits in (0, 1, 3, 8):
            desc.decode_splits = splits
            ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
            out = torch.full((S, Hq, D), 7.0, dtype=DTYPES[dt], device=DEV)
            pe.pe_paged_decode(desc, qd, kd, vd, td, ld, D ** -0.5, out, ws)
            torch.cuda.synchronize()
            got = f32(out)
            assert np.all(got[0] == 0.0), "empty sequence must give zeros"
            e2, emax = rel_err(got[1:], want[1:])
            assert e2 <= TOL[dt] and emax <= TOL[dt], (splits, e2, emax)
    finally:
        desc.decode_splits = 0


def test_paged_decode_masks_junk_and_extreme_logits():
    print("case paged_decode_masks_junk", flush=True)
    Hk, G, D, B = 2, 4, 128, 16
    lens = [21, 300]
    k_pool, v_pool, table, sl = make_paged(500, lens, Hk, D, B, torch.float32)
    # non-finite junk behind the end of every tail page must not leak in
    for s, L in enumerate(lens):
        for h in range(Hk):
            p = int(table[s, h, L // B])
            k_pool[p, L % B:] = float("nan")
            v_pool[p, L % B:] = float("inf")
    g = torch.Generator().manual_seed(501)
    q = torch.randn((2, Hk * G, D), generator=g) * 6.0      # sharp softmax: large logit spread
    want = oracle.paged_decode(f32(q), np.nan_to_num(f32(k_pool), nan=0.0, posinf=0.0),
                               np.nan_to_num(f32(v_pool), nan=0.0, posinf=0.0), i32(table), i32(sl))
    desc = pe.make_desc(torch.float32, 2, Hk, Hk * G, D, B, table.shape[2], k_pool.shape[0])
    out = torch.empty((2, Hk * G, D), dtype=torch.float32, device=DEV)
    ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
    pe.pe_paged_decode(desc, q.to(DEV), k_pool.to(DEV), v_pool.to(DEV), table.to(DEV), sl.to(DEV), D ** -0.5, out, ws)
    torch.cuda.synchronize()
    got = f32(out)
    assert np.all(np.isfinite(got))
    e2, emax = rel_err(got, want)
    assert e2 <= 1e-5 and emax <= 1e-5, (e2, emax)


@pytest.mark.parametrize("D,B", [(64, 16), (128, 16), (64, 32), (128, 64)])
@pytest.mark.parametrize("G", [1, 4, 5, 8])
def test_paged_decode_bf16_tiles(D, B, G):
    """The bf16 kernel at the edges of its tiles (16 tokens) and rounds (64 tokens, 128 with two tiles in flight), with
    non-finite junk behind every row's end and in page 0, which the kernel reads for entries a row does not use; the
    logits climb along the row, so the softmax reference has to move in later tiles; the second call writes to an output
    that is aligned to two bytes only.  Tolerance: the rounding of the
    bf16 result is 2^-9 of a value; twice that in the 2-norm, and in the max-norm of a vector."""
    print("case paged_decode_bf16_tiles", D, B, G, flush=True)
    Hk = 3
    lens = [1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 513, 1025]
    k_pool, v_pool, table, sl = make_paged(1700 + D + B + G, lens, Hk, D, B, torch.bfloat16)
    # one page more in front: page 0 is nobody's
    k_pool, v_pool = torch.cat([k_pool[:1], k_pool]), torch.cat([v_pool[:1], v_pool])
    table = torch.where(table >= 0, table + 1, table)
    P = k_pool.shape[0]
    g = torch.Generator().manual_seed(1701)
    S, Hq = len(lens), Hk * G
    q = torch.randn((S, Hq, D), generator=g)
    for s, L in enumerate(lens):   # head 0 of each group sees logits that grow with the position
        for h in range(Hk):
            for j in range((L + B - 1) // B):
                pos = torch.arange(j * B, j * B + B, dtype=torch.float32)
                u = q[s, h * G] / q[s, h * G].norm()
                k_pool[int(table[s, h, j])] += (0.02 * pos[:, None] * u[None]).to(torch.bfloat16)
    k_clean, v_clean = k_pool.clone(), v_pool.clone()
    for s, L in enumerate(lens):
        for h in range(Hk):
            if L % B:
                p = int(table[s, h, L // B])
                k_pool[p, L % B:], v_pool[p, L % B:] = float("nan"), float("inf")
    k_pool[0], v_pool[0] = float("nan"), float("-inf")
    q = q.to(torch.bfloat16)
    want = oracle.paged_decode(f32(q), f32(k_clean), f32(v_clean), i32(table), i32(sl))
    desc = pe.make_desc(torch.bfloat16, S, Hk, Hq, D, B, table.shape[2], P)
    kd, vd, td, ld, qd = (x.contiguous().to(DEV) for x in (k_pool, v_pool, table, sl, q))
    for splits in (0, 1, 2, 7):
        desc.decode_splits = splits
        ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
        for call in range(2):
            out = torch.full((S * Hq * D + 1,), 7.0, dtype=torch.bfloat16, device=DEV)[call:call + S * Hq * D].view(S, Hq, D)
            pe.pe_paged_decode(desc, qd, kd, vd, td, ld, D ** -0.5, out, ws)
            torch.cuda.synchronize()
            e2, emax = rel_err(f32(out), want)
            assert e2 <= 2 ** -8 and emax <= 2 ** -8, (splits, call, e2, emax)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G,splits", [(1, 1), (4, 2), (5, 1), (8, 2)])
def test_paged_decode_bf16_large_values(D, G, splits):
    """Values of V near the end of the range: the logit of a wave's second tile exceeds its first one's by 2.8 (base 2), and
    a weight of 2^2.8 times 1.5 * 2^126 would leave it, while the weighted sum relative to the larger logit, 1.14 of it,
    does not.  Both V are equal and all other weights 0, so the result is that value (within twice the rounding of the
    bf16 result, 2^-9)."""
    print("case paged_decode_bf16_large_values", D, G, splits, flush=True)
    B, L, big = 16, 300, 1.5 * 2.0 ** 126
    k_pool, v_pool, table, sl = make_paged(1750 + D, [L], 1, D, B, torch.bfloat16)
    v_pool.fill_(0.0)
    k_pool.fill_(0.0)
    k_pool[..., 0] = -1000.0                 # no weight
    q = torch.zeros((1, G, D))
    q[..., 0] = 8.0
    step = 2.8 / (8.0 * D ** -0.5 * 1.4426950408889634)
    for t, x in ((0, 0.0), (16 * 4 * splits, step)):   # the first tokens of the first wave's first and second tile
        page = int(table[0, 0, t // B])
        k_pool[page, t % B, 0], v_pool[page, t % B] = x, big
    desc = pe.make_desc(torch.bfloat16, 1, 1, G, D, B, table.shape[2], k_pool.shape[0])
    desc.decode_splits = splits
    out = torch.full((1, G, D), 7.0, dtype=torch.bfloat16, device=DEV)
    pe.pe_paged_decode(desc, q.to(torch.bfloat16).to(DEV), k_pool.to(DEV), v_pool.to(DEV), table.to(DEV), sl.to(DEV),
                       D ** -0.5, out, pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc))
    torch.cuda.synchronize()
    got = f32(out)
    assert np.all(np.isfinite(got))
    assert np.abs(got / big - 1.0).max() <= 2 ** -8


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_paged_decode_with_a_smaller_workspace(dt):
    """An automatic split count falls back to what the caller's workspace holds, down to splits of 256 tokens."""
    print("case paged_decode_smaller_workspace", dt, flush=True)
    Hk, G, D, B = 4, 2, 128, 16
    lens = [2048, 700, 0, 1]
    k_pool, v_pool, table, sl = make_paged(1800, lens, Hk, D, B, DTYPES[dt], extra=0)
    q = torch.randn((len(lens), Hk * G, D), generator=torch.Generator().manual_seed(1801)).to(DTYPES[dt])
    want = oracle.paged_decode(f32(q), f32(k_pool), f32(v_pool), i32(table), i32(sl))
    desc = pe.make_desc(DTYPES[dt], len(lens), Hk, Hk * G, D, B, table.shape[2], k_pool.shape[0])
    per_split = len(lens) * Hk * G * (D + 2) * 4
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("counts below are those of 256 compute units")
    assert pe.pe_decode_splits(desc) == 16
    args = [x.to(DEV) for x in (q, k_pool, v_pool, table, sl)]
    for splits in (16, 11, 8, 7):
        out = torch.full(q.shape, 7.0, dtype=DTYPES[dt], device=DEV)
        ws = torch.empty(per_split * splits, dtype=torch.uint8, device=DEV)
        if splits < 8:
            with pytest.raises(pe.PeError):
                pe.pe_paged_decode(desc, *args, D ** -0.5, out, ws)
            continue
        pe.pe_paged_decode(desc, *args, D ** -0.5, out, ws)
        torch.cuda.synchronize()
        assert np.all(f32(out)[2] == 0.0)
        live = [0, 1, 3]
        e2, emax = rel_err(f32(out)[live], want[live])
        assert e2 <= TOL[dt] and emax <= TOL[dt], (splits, e2, emax)


def _prompt(seed, lens, Hk, D, dtype, ties=False):
    g = torch.Generator().manual_seed(seed)
    T = sum(lens)
    k = (torch.randn((T, Hk, D), generator=g) * torch.exp(0.5 * torch.randn((T, Hk, 1), generator=g))).to(dtype)
    v = (torch.randn((T, Hk, D), generator=g) * torch.exp(0.5 * torch.randn((T, Hk, 1), generator=g))).to(dtype)
    if ties:   # repeat a handful of rows many times: exact score ties, also at the cut
        src = torch.randint(0, T, (T,), generator=g) % 7
        k, v = k[src].contiguous(), v[src].contiguous()
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    return k, v, cu


def _prune_both(k, v, cu, lens, Hk, D, B, C, dtype, seed):
    S = len(lens)
    need = [(min(L, C) + B - 1) // B for L in lens]
    mb = max(max(need), 1) + 1
    P = Hk * sum(need) + 2
    ids = torch.randperm(P, generator=torch.Generator().manual_seed(seed)).to(torch.int32)
    table = torch.full((S, Hk, mb), -1, dtype=torch.int32)
    pos = 0
    for s in range(S):
        for h in range(Hk):
            table[s, h, :need[s]] = ids[pos:pos + need[s]]
            pos += need[s]
    kp = np.zeros((P, B, D), np.float32); vp = np.zeros((P, B, D), np.float32)
    o_lens, o_kept = oracle.prefill_prune(f32(k), f32(v), i32(cu), C, kp, vp, i32(table))
    desc = pe.make_desc(dtype, S, Hk, Hk, D, B, mb, P)
    kpd = torch.zeros((P, B, D), dtype=dtype, device=DEV); vpd = torch.zeros((P, B, D), dtype=dtype, device=DEV)
    lens_d = torch.full((S,), -5, dtype=torch.int32, device=DEV)
    kept_d = torch.full((S, Hk, C), -9, dtype=torch.int32, device=DEV)
    ws = pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, int(cu[-1]))
    pe.pe_prefill_prune(desc, k.to(DEV), v.to(DEV), cu.to(DEV), int(cu[-1]), max(lens), C, kpd, vpd, table.to(DEV),
                        lens_d, kept_d, ws)
    torch.cuda.synchronize()
    assert np.array_equal(lens_d.cpu().numpy(), o_lens)
    assert np.array_equal(kept_d.cpu().numpy(), o_kept)
    # pool contents: every slot the oracle wrote (the rest stayed zero on both sides)
    assert np.array_equal(f32(kpd).view(np.int32), kp.view(np.int32))
    assert np.array_equal(f32(vpd).view(np.int32), vp.view(np.int32))
    return o_kept


@pytest.mark.parametrize("dt,D", [("f32", 64), ("bf16", 64), ("bf16", 128), ("f32", 128)])
def test_prefill_prune_ragged(dt, D):
    print("case prefill_prune_ragged", dt, D, flush=True)
    lens = [1, 100, 1023, 1024, 1025, 3000, 5000, 256]
    for C, B in ((256, 16), (1024, 32), (512, 64), (1024, 128)):
        k, v, cu = _prompt(600 + D + C, lens, 2, D, DTYPES[dt])
        _prune_both(k, v, cu, lens, 2, D, B, C, DTYPES[dt], 601)


def test_prefill_prune_ties():
    print("case prefill_prune_ties", flush=True)
    lens = [2100, 700]
    k, v, cu = _prompt(610, lens, 2, 128, torch.bfloat16, ties=True)
    kept = _prune_both(k, v, cu, lens, 2, 128, 16, 512, torch.bfloat16, 611)
    assert kept.max() > 0
    # V = K: every score is exactly 1 -> the E lowest indices go
    kept = _prune_both(k, k.clone(), cu, lens, 2, 128, 16, 512, torch.bfloat16, 612)
    assert np.array_equal(kept[0, 0], np.arange(2100 - 512, 2100))


@pytest.mark.parametrize("lens", [[1, 4095, 3], [4096, 2, 4097], [6, 8191, 8193], [1, 16383, 16385], [2, 32768],
                                  [32769, 5], [1, 33793, 32767], [3, 66000], [32770, 1, 49151], [32771, 49153],
                                  [2, 49155, 65541]])
@pytest.mark.parametrize("crowded", [False, True])
def test_prefill_prune_row_holding(lens, crowded):
    """Rows at the edges of what the selection holds in registers (4096 * 1, 2, 4, 8 scores) and beyond, starting
    at offsets that are not multiples of four scores; crowded: scores with so few distinct values that the threshold
    bin overflows the candidate list and many scores tie at the cut.  Integers and copies: bit for bit."""
    print("case prefill_prune_row_holding", lens, crowded, flush=True)
    k, v, cu = _prompt(640 + len(lens), lens, 1, 64, torch.bfloat16, ties=crowded)
    _prune_both(k, v, cu, lens, 1, 64, 16, 1024, torch.bfloat16, 641)


def test_prefill_prune_crowded_threshold_bin():
    """Rows whose scores crowd into one bin of the selection's first radix digit, more of them than its LDS
    candidate buffer holds (8192): the later digits are then resolved by passes over memory.  (a) all scores equal
    (V = K), rows of 20000 and 9001 tokens starting at offsets that are not multiples of four scores; (b) fp32 rows
    with V = K * c, c spread over [1, 1.1): one first-digit bin, distinct lower digits; (c) a mix in which the
    threshold bin is crowded and other bins are populated too."""
    print("case prefill_prune_crowded_bin", flush=True)
    lens = [3, 20000, 9001, 1022]
    k, _, cu = _prompt(620, lens, 2, 64, torch.bfloat16)
    kept = _prune_both(k, k.clone(), cu, lens, 2, 64, 16, 1024, torch.bfloat16, 621)          # (a)
    assert np.array_equal(kept[1, 0], np.arange(20000 - 1024, 20000))
    assert np.array_equal(kept[2, 1], np.arange(9001 - 1024, 9001))
    g = torch.Generator().manual_seed(622)
    lens = [17000, 5]
    k, _, cu = _prompt(623, lens, 2, 64, torch.float32)
    c = 1.0 + 0.1 * torch.rand((sum(lens), 2, 1), generator=g)
    _prune_both(k, (k * c).contiguous(), cu, lens, 2, 64, 32, 2048, torch.float32, 624)       # (b)
    c[::3] = torch.exp(torch.randn((c[::3].shape[0], 2, 1), generator=g))                     # (c) a third elsewhere
    _prune_both(k, (k * c).contiguous(), cu, lens, 2, 64, 32, 4096, torch.float32, 625)


def test_append_kv_matches_oracle():
    print("case append_kv", flush=True)
    Hk, D, B = 3, 64, 16
    lens = [16, 5, 0, 31, 32]
    k_pool, v_pool, table, sl = make_paged(700, lens, Hk, D, B, torch.bfloat16, extra=2, pad_pages=40)
    S, mb, P = len(lens), table.shape[2], k_pool.shape[0]
    used = set(int(x) for x in table.flatten() if x >= 0)
    free = [p for p in range(P) if p not in used]
    n_spare = 2
    spare = torch.tensor(free[:S * Hk * n_spare], dtype=torch.int32).reshape(S, Hk, n_spare)
    freed = torch.full((S, Hk), -1, dtype=torch.int32)
    freed[0, 1] = free[-1]                         # one row re-uses a page it "just freed"
    spare_used = torch.zeros((S, Hk), dtype=torch.int32)
    o = dict(k=f32(k_pool), v=f32(v_pool), t=i32(table).copy(), l=i32(sl).copy(), f=i32(freed).copy(),
             u=i32(spare_used).copy())
    desc = pe.make_desc(torch.bfloat16, S, Hk, Hk, D, B, mb, P)
    kd, vd, td, ld, fd, sd, ud = (x.to(DEV) for x in (k_pool, v_pool, table, sl, freed, spare, spare_used))
    g = torch.Generator().manual_seed(701)
    for step in range(3):
        nk = torch.randn((S, Hk, D), generator=g).to(torch.bfloat16)
        nv = torch.randn((S, Hk, D), generator=g).to(torch.bfloat16)
        oracle.append_kv(f32(nk), f32(nv), o["k"], o["v"], o["t"], o["l"], o["f"], i32(spare), o["u"])
        pe.pe_append_kv(desc, nk.to(DEV), nv.to(DEV), kd, vd, td, ld, fd, sd, ud)
        torch.cuda.synchronize()
        assert np.array_equal(td.cpu().numpy(), o["t"]) and np.array_equal(ld.cpu().numpy(), o["l"])
        assert np.array_equal(fd.cpu().numpy(), o["f"]) and np.array_equal(ud.cpu().numpy(), o["u"])
        assert np.array_equal(f32(kd).view(np.int32), o["k"].view(np.int32))
        assert np.array_equal(f32(vd).view(np.int32), o["v"].view(np.int32))


@pytest.mark.parametrize("dt,D,B,G", [("bf16", 128, 16, 4), ("bf16", 64, 16, 4), ("f32", 64, 16, 2), ("bf16", 128, 32, 3),
                                      ("f32", 128, 32, 1), ("bf16", 64, 32, 8), ("bf16", 128, 64, 4),
                                      ("f32", 64, 128, 2)])
def test_append_paged_decode_fused(dt, D, B, G):
    """The one-launch append + attention against the oracle's append followed by its attention, three
    steps in a row: tables, lengths, spare/freed bookkeeping and pool contents bit-exact, output in
    tolerance.  Rows at a page boundary take a freed page or a spare one; one sequence is empty."""
    print("case append_paged_decode_fused", dt, D, B, G, flush=True)
    Hk = 2
    lens = [0, 1, B - 1, B, 2 * B, 5 * B + 3, 40 * B, 40 * B - 1, 1300]
    k_pool, v_pool, table, sl = make_paged(800 + D + B + G, lens, Hk, D, B, DTYPES[dt], extra=2, pad_pages=64)
    S, Hq, mb, P = len(lens), Hk * G, table.shape[2], k_pool.shape[0]
    used = set(int(x) for x in table.flatten() if x >= 0)
    free = [p for p in range(P) if p not in used]
    n_spare = 2
    spare = torch.tensor(free[:S * Hk * n_spare], dtype=torch.int32).reshape(S, Hk, n_spare)
    freed = torch.full((S, Hk), -1, dtype=torch.int32)
    freed[3, 0] = free[-1]            # sequence 3 (len == B) re-uses a "freed" page in head 0, a spare in head 1
    freed[6, 1] = free[-2]
    spare_used = torch.zeros((S, Hk), dtype=torch.int32)
    o = dict(k=f32(k_pool), v=f32(v_pool), t=i32(table).copy(), l=i32(sl).copy(), f=i32(freed).copy(),
             u=i32(spare_used).copy())
    desc = pe.make_desc(DTYPES[dt], S, Hk, Hq, D, B, mb, P)
    kd, vd, td, ld, fd, sd, ud = (x.to(DEV) for x in (k_pool, v_pool, table, sl, freed, spare, spare_used))
    g = torch.Generator().manual_seed(801)
    try:
        for step, splits in enumerate((1, 3, 0)):
            desc.decode_splits = splits
            ws = pe.alloc_workspace(pe.PE_OP_APPEND_PAGED_DECODE, desc)
            nk = torch.randn((S, Hk, D), generator=g).to(DTYPES[dt])
            nv = torch.randn((S, Hk, D), generator=g).to(DTYPES[dt])
            q = torch.randn((S, Hq, D), generator=g).to(DTYPES[dt])
            oracle.append_kv(f32(nk), f32(nv), o["k"], o["v"], o["t"], o["l"], o["f"], i32(spare), o["u"])
            want = oracle.paged_decode(f32(q), o["k"], o["v"], o["t"], o["l"])
            out = torch.full((S, Hq, D), 7.0, dtype=DTYPES[dt], device=DEV)
            for rep in range(1):
                ld_out = torch.full_like(ld, -3)
                pe.pe_append_paged_decode(desc, nk.to(DEV), nv.to(DEV), q.to(DEV), kd, vd, td, ld, ld_out, fd, sd, ud,
                                          D ** -0.5, out, ws)
                torch.cuda.synchronize()
                ld = ld_out
                assert np.array_equal(td.cpu().numpy(), o["t"]) and np.array_equal(ld.cpu().numpy(), o["l"])
                assert np.array_equal(fd.cpu().numpy(), o["f"]) and np.array_equal(ud.cpu().numpy(), o["u"])
                assert np.array_equal(f32(kd).view(np.int32), o["k"].view(np.int32))
                assert np.array_equal(f32(vd).view(np.int32), o["v"].view(np.int32))
                e2, emax = rel_err(f32(out), want)
                assert e2 <= TOL[dt] and emax <= TOL[dt], (step, rep, e2, emax)
    finally:
        desc.decode_splits = 0


@pytest.mark.parametrize("D,B,lens", [(64, 16, [1, 15, 16, 17, 33, 63, 64, 65, 129, 300, 511, 513, 1000]),
                                      (64, 64, [1, 63, 64, 65, 191, 575]), (128, 16, [1, 7, 8, 9, 16, 31, 33, 65, 127, 150]),
                                      (128, 32, [1, 32, 33, 95, 128])])
def test_bf16_short_rows_of_one_head(D, B, lens):
    """Short rows of one query head per KV head, at the edges of tiles (8 and 16 tokens) and rounds, with non-finite junk behind
    every row's end: attention, and the append in the same launch, whole and in splits.  Tolerance: twice the rounding of the
    bf16 result, 2^-9."""
    print("case bf16_short_rows_of_one_head", D, B, flush=True)
    Hk = 3
    k_pool, v_pool, table, sl = make_paged(1970 + D + B, lens, Hk, D, B, torch.bfloat16, pad_pages=len(lens) * Hk)
    S, mb, P = len(lens), table.shape[2], k_pool.shape[0]
    assert mb * B <= (1024 if D == 64 else 192)   # tables that lead to the vector units
    for s, L in enumerate(lens):
        if L % B:
            for p in table[s, :, L // B].tolist():
                k_pool[p, L % B:], v_pool[p, L % B:] = float("nan"), float("inf")
    clean = lambda t: np.nan_to_num(f32(t), nan=0.0, posinf=0.0)
    used = set(table[table >= 0].tolist())
    spare = torch.tensor([p for p in range(P) if p not in used], dtype=torch.int32).reshape(S, Hk, 1)
    g = torch.Generator().manual_seed(1971)
    q = torch.randn((S, Hk, D), generator=g).to(torch.bfloat16)
    nk, nv = (torch.randn((S, Hk, D), generator=g).to(torch.bfloat16) for _ in range(2))
    o = dict(k=clean(k_pool), v=clean(v_pool), t=i32(table).copy(), l=i32(sl).copy())
    want = [oracle.paged_decode(f32(q), o["k"], o["v"], o["t"], o["l"])]
    oracle.append_kv(f32(nk), f32(nv), o["k"], o["v"], o["t"], o["l"], np.full((S, Hk), -1, np.int32), i32(spare),
                     np.zeros((S, Hk), np.int32))
    want.append(oracle.paged_decode(f32(q), o["k"], o["v"], o["t"], o["l"]))
    for splits in (0, 1, 3):
        desc = pe.make_desc(torch.bfloat16, S, Hk, Hk, D, B, mb, P, decode_splits=splits)
        ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
        qd, kd, vd, td, ld, sd, nkd, nvd = (x.to(DEV) for x in (q, k_pool, v_pool, table, sl, spare, nk, nv))
        fd, ud = (torch.full((S, Hk), x, dtype=torch.int32, device=DEV) for x in (-1, 0))
        outs = [torch.full(q.shape, 7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
        ld_out = torch.full_like(ld, -3)
        pe.pe_paged_decode(desc, qd, kd, vd, td, ld, D ** -0.5, outs[0], ws)
        pe.pe_append_paged_decode(desc, nkd, nvd, qd, kd, vd, td, ld, ld_out, fd, sd, ud, D ** -0.5, outs[1], ws)
        torch.cuda.synchronize()
        for out, w in zip(outs, want):
            e2, emax = rel_err(f32(out), w)
            assert e2 <= 2 ** -8 and emax <= 2 ** -8, (splits, e2, emax)
        assert np.array_equal(td.cpu().numpy(), o["t"]) and np.array_equal(ld_out.cpu().numpy(), o["l"])
        assert np.array_equal(clean(kd), o["k"]) and np.array_equal(clean(vd), o["v"])


@pytest.mark.parametrize("shape", [422, 424, 432, 822])
def test_bf16_named_shapes(shape):
    """The workgroup forms that a descriptor can name, at the edges of their tiles and rounds: attention, and the append in
    the same launch.  Tolerance: twice the rounding of the bf16 result, 2^-9."""
    print("case bf16_named_shapes", shape, flush=True)
    D, B, Hk, G = 128, 16, 2, 4
    lens = [1, 15, 16, 17, 63, 64, 65, 127, 129, 191, 193, 255, 256, 257, 385, 513, 1025]
    k_pool, v_pool, table, sl = make_paged(1950, lens, Hk, D, B, torch.bfloat16, pad_pages=len(lens) * Hk)
    S, mb, P = len(lens), table.shape[2], k_pool.shape[0]
    used = set(table[table >= 0].tolist())
    spare = torch.tensor([p for p in range(P) if p not in used], dtype=torch.int32).reshape(S, Hk, 1)
    g = torch.Generator().manual_seed(1951)
    q = torch.randn((S, Hk * G, D), generator=g).to(torch.bfloat16)
    nk, nv = (torch.randn((S, Hk, D), generator=g).to(torch.bfloat16) for _ in range(2))
    o = dict(k=f32(k_pool).copy(), v=f32(v_pool).copy(), t=i32(table).copy(), l=i32(sl).copy())
    want = [oracle.paged_decode(f32(q), o["k"], o["v"], o["t"], o["l"])]
    oracle.append_kv(f32(nk), f32(nv), o["k"], o["v"], o["t"], o["l"], np.full((S, Hk), -1, np.int32), i32(spare),
                     np.zeros((S, Hk), np.int32))
    want.append(oracle.paged_decode(f32(q), o["k"], o["v"], o["t"], o["l"]))
    for splits in (1, 3):
        desc = pe.make_desc(torch.bfloat16, S, Hk, Hk * G, D, B, mb, P, decode_splits=splits, decode_shape=shape)
        ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
        qd, kd, vd, td, ld, sd, nkd, nvd = (x.to(DEV) for x in (q, k_pool, v_pool, table, sl, spare, nk, nv))
        fd, ud = (torch.full((S, Hk), x, dtype=torch.int32, device=DEV) for x in (-1, 0))
        outs = [torch.full(q.shape, 7.0, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
        ld_out = torch.full_like(ld, -3)
        pe.pe_paged_decode(desc, qd, kd, vd, td, ld, D ** -0.5, outs[0], ws)
        pe.pe_append_paged_decode(desc, nkd, nvd, qd, kd, vd, td, ld, ld_out, fd, sd, ud, D ** -0.5, outs[1], ws)
        torch.cuda.synchronize()
        for out, w in zip(outs, want):
            e2, emax = rel_err(f32(out), w)
            assert e2 <= 2 ** -8 and emax <= 2 ** -8, (splits, e2, emax)
        assert np.array_equal(td.cpu().numpy(), o["t"]) and np.array_equal(ld_out.cpu().numpy(), o["l"])
        assert np.array_equal(f32(kd), o["k"]) and np.array_equal(f32(vd), o["v"])


@pytest.mark.parametrize("D,G", [(128, 1), (128, 4), (128, 5), (128, 8), (64, 4), (64, 8)])
@pytest.mark.parametrize("fused", [False, True])
def test_bf16_row_for_every_compute_unit(D, G, fused):
    """As many rows as compute units in table rows of 2048 tokens, which the rows fill in part: whole rows of D = 128 run in
    workgroups of eight waves (tiles in rounds of 128 tokens, 256 with two in flight); in two splits each, workgroups with one
    tile in flight share a compute unit.  Lengths at the edges of tiles and rounds; attention alone, and with the append.  Tolerance: twice the
    rounding of the bf16 result, 2^-9."""
    print("case bf16_row_for_every_compute_unit", D, G, fused, flush=True)
    B, Hk = 16, 8
    S = torch.cuda.get_device_properties(0).multi_processor_count // Hk
    edges = [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 143, 144, 255, 256, 257, 383, 384, 511, 513, 1025]
    lens = [edges[s % len(edges)] for s in range(S)]
    k_pool, v_pool, table, sl = make_paged(1900 + G, lens, Hk, D, B, torch.bfloat16, extra=2048 // B - 65, pad_pages=S * Hk)
    P, mb = k_pool.shape[0], table.shape[2]
    assert mb * B == 2048
    for s, L in enumerate(lens):   # junk behind the end of a tail page
        if L % B:
            for p in table[s, :, L // B].tolist():
                k_pool[p, L % B:], v_pool[p, L % B:] = float("nan"), float("inf")
    clean = lambda t: np.nan_to_num(f32(t), nan=0.0, posinf=0.0)
    used = set(table[table >= 0].tolist())
    spare = torch.tensor([p for p in range(P) if p not in used], dtype=torch.int32).reshape(S, Hk, 1)
    o = dict(k=clean(k_pool), v=clean(v_pool), t=i32(table).copy(), l=i32(sl).copy(), f=np.full((S, Hk), -1, np.int32),
             u=np.zeros((S, Hk), np.int32))
    g = torch.Generator().manual_seed(1901)
    kd, vd, td, ld, sd = (x.to(DEV) for x in (k_pool, v_pool, table, sl, spare))
    fd, ud = torch.from_numpy(o["f"]).to(DEV), torch.from_numpy(o["u"]).to(DEV)
    for splits in (1, 2):
        desc = pe.make_desc(torch.bfloat16, S, Hk, Hk * G, D, B, mb, P)
        desc.decode_splits = splits
        ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
        q = torch.randn((S, Hk * G, D), generator=g).to(torch.bfloat16)
        out = torch.full(q.shape, 7.0, dtype=torch.bfloat16, device=DEV)
        if fused:
            nk, nv = (torch.randn((S, Hk, D), generator=g).to(torch.bfloat16) for _ in range(2))
            oracle.append_kv(f32(nk), f32(nv), o["k"], o["v"], o["t"], o["l"], o["f"], i32(spare), o["u"])
            ld_out = torch.full_like(ld, -3)
            pe.pe_append_paged_decode(desc, nk.to(DEV), nv.to(DEV), q.to(DEV), kd, vd, td, ld, ld_out, fd, sd, ud, D ** -0.5,
                                      out, ws)
            ld = ld_out
        else:
            pe.pe_paged_decode(desc, q.to(DEV), kd, vd, td, ld, D ** -0.5, out, ws)
        torch.cuda.synchronize()
        want = oracle.paged_decode(f32(q), o["k"], o["v"], o["t"], o["l"])
        e2, emax = rel_err(f32(out), want)
        assert e2 <= 2 ** -8 and emax <= 2 ** -8, (splits, e2, emax)
        assert np.array_equal(td.cpu().numpy(), o["t"]) and np.array_equal(ld.cpu().numpy(), o["l"])
        assert np.array_equal(ud.cpu().numpy(), o["u"])
        for s in range(S):   # the stored rows
            n = int(o["l"][s])
            p = o["t"][s, :, (n - 1) // B]
            assert np.array_equal(f32(kd[p, (n - 1) % B]), o["k"][p, (n - 1) % B])
            assert np.array_equal(f32(vd[p, (n - 1) % B]), o["v"][p, (n - 1) % B])


@pytest.mark.parametrize("opts", [dict(policy=0, protect_first=2, protect_last=3), dict(policy=1, protect_first=4),
                                  dict(policy=0, share_heads=True), dict(policy=0, share_heads=True, protect_first=1),
                                  dict(policy=1), dict(policy=0, protect_first=500)])
@pytest.mark.parametrize("cached", [False, True])
def test_evict_blocks_ex_bit_exact(opts, cached):
    """Eviction variants against the oracle on rows of 1 .. 300 pages with many tied scores; with cached
    scores the score rows must be compacted exactly like the table rows."""
    print("case evict_blocks_ex", opts, cached, flush=True)
    rng = np.random.default_rng(900)
    B, Hk = 16, 6
    n_pages = [1, 2, 5, 63, 64, 65, 129, 300, 7, 40, 0]
    S, mb = len(n_pages), 301
    lens = np.array([n * B for n in n_pages], np.int32)
    lens[8] -= 5
    C = 2 * B
    scores = (rng.integers(0, 6, size=(S, Hk, mb)) * 0.25 + rng.integers(0, 2, size=(S, Hk, mb)) * 2.0 ** -20
              ).astype(np.float32)
    table = np.full((S, Hk, mb), -1, np.int32)
    ids = rng.permutation(S * Hk * mb).astype(np.int32)
    pos = 0
    for s in range(S):
        n = (lens[s] + B - 1) // B
        for h in range(Hk):
            table[s, h, :n] = ids[pos:pos + n]
            pos += n
    desc = pe.make_desc(torch.float32, S, Hk, Hk, 64, B, mb, S * Hk * mb)
    o = pe.pe_evict_opts(opts.get("policy", 0), opts.get("protect_first", 0), opts.get("protect_last", 0),
                         int(opts.get("share_heads", False)), int(cached))
    t_gpu, l_gpu = torch.tensor(table, device=DEV), torch.tensor(lens, device=DEV)
    s_gpu = torch.tensor(scores, device=DEV)
    ev_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    fr_gpu = torch.full((S, Hk), -7, dtype=torch.int32, device=DEV)
    sc = scores.copy()
    for call in range(3):
        n_before = lens // B
        ev, fr = oracle.evict_blocks_ex(sc, table, lens, B, C, **opts)
        pe.pe_evict_blocks_ex(desc, o, None if (opts.get("policy", 0) == 1 and not cached) else s_gpu, t_gpu, l_gpu, C,
                              ev_gpu, fr_gpu)
        torch.cuda.synchronize()
        assert np.array_equal(ev_gpu.cpu().numpy(), ev), call
        assert np.array_equal(fr_gpu.cpu().numpy(), fr), call
        assert np.array_equal(t_gpu.cpu().numpy(), table), call
        assert np.array_equal(l_gpu.cpu().numpy(), lens), call
        if cached:      # delete the evicted entry from the reference score rows as well
            for s in range(S):
                for h in range(Hk):
                    j, n = ev[s, h], n_before[s]
                    if j >= 0:
                        sc[s, h, j:n - 1] = sc[s, h, j + 1:n].copy()
                        sc[s, h, n - 1] = np.inf
            assert np.array_equal(s_gpu.cpu().numpy().view(np.int32), sc.view(np.int32)), call
    if opts.get("share_heads"):
        trig = ev[:, 0] >= 0
        assert np.all(ev[trig] == ev[trig][:, :1])


def test_extreme_shapes_and_single_row():
    """Smallest shapes (one sequence, one KV head, one-page table), widest group (8 query heads per KV head),
    fp32 with head_dim 128 and 32-token pages (the largest register tile), many short sequences."""
    print("case extreme shapes", flush=True)
    for dt, D, B, Hk, G, lens in (("f32", 128, 32, 1, 8, [1]), ("bf16", 64, 16, 1, 1, [16]), ("f32", 64, 32, 1, 5, [31]),
                                  ("bf16", 128, 16, 3, 7, [2] * 70), ("f32", 128, 32, 2, 8, [97, 3000])):
        extra = 0 if len(lens) == 1 else 1
        k_pool, v_pool, table, sl = make_paged(950 + D + B + G, lens, Hk, D, B, DTYPES[dt], extra=extra)
        S, Hq, mb, P = len(lens), Hk * G, table.shape[2], k_pool.shape[0]
        g = torch.Generator().manual_seed(951)
        q = torch.randn((S, Hq, D), generator=g).to(DTYPES[dt])
        desc = pe.make_desc(DTYPES[dt], S, Hk, Hq, D, B, mb, P)
        kd, vd, td, ld = (x.to(DEV) for x in (k_pool, v_pool, table, sl))
        # scores
        got = gpu_scores(k_pool, v_pool, table, sl, Hq)
        want = oracle.score_blocks(f32(k_pool), f32(v_pool), i32(table), i32(sl))
        assert np.array_equal(np.isinf(got), np.isinf(want))
        fin = np.isfinite(want)
        assert fin.sum() == 0 or _ulp_diff(got[fin], want[fin]).max() <= 1
        # attention
        out = torch.empty((S, Hq, D), dtype=DTYPES[dt], device=DEV)
        ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
        pe.pe_paged_decode(desc, q.to(DEV), kd, vd, td, ld, D ** -0.5, out, ws)
        torch.cuda.synchronize()
        e2, emax = rel_err(f32(out), oracle.paged_decode(f32(q), f32(k_pool), f32(v_pool), i32(table), i32(sl)))
        assert e2 <= TOL[dt] and emax <= TOL[dt], (dt, D, B, Hk, G, e2, emax)


def test_calls_run_on_the_callers_stream():
    """Every call enqueues on the stream it is given: work issued on a side stream, behind a long-running
    producer on that stream, must see the producer's result without any extra synchronisation."""
    print("case side stream", flush=True)
    Hk, G, D, B = 2, 4, 128, 16
    lens = [300, 77]
    k_pool, v_pool, table, sl = make_paged(990, lens, Hk, D, B, torch.bfloat16)
    S, Hq, mb, P = 2, Hk * G, table.shape[2], k_pool.shape[0]
    g = torch.Generator().manual_seed(991)
    q = torch.randn((S, Hq, D), generator=g).to(torch.bfloat16)
    want = oracle.paged_decode(f32(q), f32(k_pool), f32(v_pool), i32(table), i32(sl))
    desc = pe.make_desc(torch.bfloat16, S, Hk, Hq, D, B, mb, P)
    kd, vd, td, ld = (x.to(DEV) for x in (k_pool, v_pool, table, sl))
    ws = pe.alloc_workspace(pe.PE_OP_PAGED_DECODE, desc)
    side = torch.cuda.Stream()
    qd = torch.zeros((S, Hq, D), dtype=torch.bfloat16, device=DEV)
    out = torch.empty_like(qd)
    scores = torch.empty((S, Hk, mb), dtype=torch.float32, device=DEV)
    big = torch.empty(1 << 28, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(8):
            big.fill_(1)                      # keeps the side stream busy for a while
        qd.copy_(q.to(DEV, non_blocking=True))   # the query only becomes valid on this stream, after the fills
        pe.pe_paged_decode(desc, qd, kd, vd, td, ld, D ** -0.5, out, ws)
        pe.pe_score_blocks(desc, kd, vd, td, ld, scores)
    side.synchronize()
    e2, emax = rel_err(f32(out), want)
    assert e2 <= 2e-2 and emax <= 2e-2
    assert np.array_equal(np.isinf(scores.cpu().numpy()),
                          np.isinf(oracle.score_blocks(f32(k_pool), f32(v_pool), i32(table), i32(sl))))
