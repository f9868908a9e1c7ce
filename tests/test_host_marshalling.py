"""The native argument marshalling: what it takes, what it leaves to the way through ctypes (which accepts it or says what is
wrong), and that both make the same call."""
import ctypes

import pytest
import torch

from paper_2509_04377_amd import binding as pe
from paper_2509_04377_amd import synth
from paper_2509_04377_amd.engine import LayeredCache, PagedCache

S, Hk, Hq, D, B, PAGES = 3, 2, 4, 64, 16, 4


def _args(dev):
    g = torch.Generator().manual_seed(3)
    P = S * Hk * PAGES
    k, v = (torch.randn((P, B, D), generator=g).to(dev) for _ in range(2))
    table = torch.arange(P, dtype=torch.int32).view(S, Hk, PAGES).to(dev)
    lens = torch.tensor([1, 40, 63], dtype=torch.int32).to(dev)
    q = torch.randn((S, Hq, D), generator=g).to(dev)
    return pe.make_desc(torch.float32, S, Hk, Hq, D, B, PAGES, P), q, k, v, table, lens


def test_what_is_not_a_dense_gpu_tensor_is_left_to_ctypes():
    L = pe.lib()
    desc, q, k, v, table, lens = _args("cpu")
    assert pe._host.paged_decode(L.addr_paged_decode, desc, q, k, v, table, lens, 0.1, q, None) is None
    with pytest.raises(ValueError, match="q must be a GPU tensor"):
        pe.pe_paged_decode(desc, q, k, v, table, lens, 0.1, torch.empty_like(q))
    with pytest.raises(TypeError):
        pe._host.paged_decode(L.addr_paged_decode, desc)
    with pytest.raises(ValueError):
        pe._host.paged_decode(0, desc, q, k, v, table, lens, 0.1, q, None)


def test_workspace_in_host_memory_is_refused():
    assert pe._ws(None) == (None, 0)
    with pytest.raises(ValueError, match="workspace must be a GPU tensor"):
        pe._ws(torch.empty(1 << 16, dtype=torch.uint8))


def test_descriptor_is_the_structure_of_the_header():
    """The extension is compiled from include/pe.h: size, and name, offset and size of every field."""
    pe.lib()
    assert ctypes.sizeof(pe.pe_cache_desc) == 56
    assert pe._host.bind_descriptor(pe.pe_cache_desc) == pe._layout(pe.pe_cache_desc)
    with pytest.raises(TypeError):
        pe._host.bind_descriptor(pe.pe_cache_desc())


class _LongerDesc(pe.pe_cache_desc):
    _fields_ = [("more", ctypes.c_int32)]


class _SameDesc(pe.pe_cache_desc):
    pass


@pytest.mark.gpu
def test_native_call_and_ctypes_call_are_the_same():
    L = pe.lib()
    desc, q, k, v, table, lens = _args("cuda")
    outs = [torch.empty_like(q) for _ in range(3)]
    assert pe._host.paged_decode(L.addr_paged_decode, desc, q, k, v, table, lens, 0.125, outs[0], None) == pe.PE_OK
    pe.pe_paged_decode(desc, q, k, v, table, lens, 0.125, outs[1])
    pe.pe_paged_decode(desc, q, k, v, table, lens, torch.tensor(0.125), outs[2])   # a scale that only float() understands
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.gpu
def test_gpu_arguments_that_are_refused():
    L = pe.lib()
    desc, q, k, v, table, lens = _args("cuda")
    out = torch.empty_like(q)
    bad = {"q": q.transpose(0, 1), "table": table.long(), "lens": lens.float()}
    assert pe._host.paged_decode(L.addr_paged_decode, desc, bad["q"], k, v, table, lens, 0.1, out, None) is None
    with pytest.raises(ValueError, match="q must be contiguous"):
        pe.pe_paged_decode(desc, bad["q"], k, v, table, lens, 0.1, out)
    with pytest.raises(ValueError, match="block_table must be torch.int32"):
        pe.pe_paged_decode(desc, q, k, v, bad["table"], lens, 0.1, out)
    with pytest.raises(ValueError, match="seq_lens must be torch.int32"):
        pe.pe_paged_decode(desc, q, k, v, table, bad["lens"], 0.1, out)
    with pytest.raises(pe.PeError):   # a status that the library gives
        pe.pe_paged_decode(pe.make_desc(torch.float32, S, Hk, Hq, 96, B, PAGES, S * Hk * PAGES), q, k, v, table, lens, 0.1, out)
    with pytest.raises(pe.PeError):
        pe.pe_paged_decode(desc, None, k, v, table, lens, 0.1, out)


@pytest.mark.gpu
def test_descriptor_of_another_type():
    """56 bytes of anything are no descriptor: what ctypes.byref refuses stays refused, what it takes (a structure derived from
    the descriptor) goes that way."""
    desc, q, k, v, table, lens = _args("cuda")
    given = []
    vp = ctypes.c_void_p
    stand_in = ctypes.CFUNCTYPE(ctypes.c_int, vp, vp, vp, vp, vp, vp, ctypes.c_float, vp, vp, ctypes.c_size_t, vp)(
        lambda *a: given.append(a) or 0)
    address = ctypes.cast(stand_in, vp).value
    raw = bytes(desc)
    values = [getattr(desc, name) for name, _ in desc._fields_]
    others = [raw, raw[:-1], bytearray(raw), memoryview(raw), (ctypes.c_char * len(raw))(*raw), torch.zeros(7), None]
    for other in others + [_LongerDesc(*values), _SameDesc(*values)]:
        assert pe._host.paged_decode(address, other, q, k, v, table, lens, 0.125, q, None) is None and not given
    assert pe._host.paged_decode(address, desc, q, k, v, table, lens, 0.125, q, None) == 0 and len(given) == 1
    want, got = torch.empty_like(q), torch.empty_like(q)
    pe.pe_paged_decode(desc, q, k, v, table, lens, 0.125, want)
    for other in others:
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            pe.pe_paged_decode(other, q, k, v, table, lens, 0.125, got)
    for other in (_LongerDesc(*values), _SameDesc(*values)):
        pe.pe_paged_decode(other, q, k, v, table, lens, 0.125, got.zero_())
        assert torch.equal(want, got)


@pytest.mark.gpu
def test_workspace_that_is_not_a_dense_gpu_tensor():
    """What a workspace claims to hold has to be device memory of its own.  The native call gets a stand-in for the C function:
    nothing is launched with any of these."""
    desc, q, k, v, table, lens = _args("cuda")
    desc.decode_splits = 4
    need = pe.pe_workspace_bytes(pe.PE_OP_PAGED_DECODE, desc)
    given = []
    vp = ctypes.c_void_p
    stand_in = ctypes.CFUNCTYPE(ctypes.c_int, vp, vp, vp, vp, vp, vp, ctypes.c_float, vp, vp, ctypes.c_size_t, vp)(
        lambda *a: given.append((a[8], a[9])) or 0)
    address = ctypes.cast(stand_in, vp).value
    whole = torch.empty((2, need), dtype=torch.uint8, device="cuda")
    bad = {"host": torch.empty(need, dtype=torch.uint8), "gaps": whole.view(-1)[::2], "columns": whole[:, :need // 2],
           "repeated": whole[0, :1].expand(need), "sparse": torch.zeros((4, need), device="cuda").to_sparse()}
    for kind, ws in bad.items():
        assert pe._host.paged_decode(address, desc, q, k, v, table, lens, 0.125, q, ws) is None and not given, kind
    for kind, ws in bad.items():
        if kind != "sparse":
            with pytest.raises(ValueError, match="workspace must be"):
                pe.pe_paged_decode(desc, q, k, v, table, lens, 0.125, torch.empty_like(q), ws)
    for ws in (whole, whole[1], whole.t(), None):
        assert pe._host.paged_decode(address, desc, q, k, v, table, lens, 0.125, q, ws) == 0
        assert pe._ws(ws) == given[-1]


@pytest.mark.gpu
def test_native_call_runs_on_the_current_stream():
    desc, q, k, v, table, lens = _args("cuda")
    want, got = torch.empty_like(q), torch.zeros_like(q)
    pe.pe_paged_decode(desc, q, k, v, table, lens, 0.125, want)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        scratch = torch.randn((2048, 2048), device="cuda")
        for _ in range(20):
            scratch = scratch @ scratch / 2048
        late = q + 0 * scratch[0, 0]
        pe.pe_paged_decode(desc, late, k, v, table, lens, 0.125, got)   # behind `late` only on this stream
    side.synchronize()
    assert torch.equal(got, want)


@pytest.mark.gpu
def test_score_and_evict_marshalling():
    L = pe.lib()
    desc, q, k, v, table, lens = _args("cuda")
    lens = torch.tensor([16, 64, 48], dtype=torch.int32, device="cuda")
    outs = []
    for native in (True, False):
        t, n = table.clone(), lens.clone()
        scores = torch.zeros((S, Hk, PAGES), device="cuda")
        gone, freed = (torch.full((S, Hk), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        budget = 48 if native else torch.tensor(48)   # only int() understands the second
        if native:
            assert pe._host.score_triggered_blocks(L.addr_score_triggered_blocks, desc, k, v, t, n, budget, scores) == pe.PE_OK
            assert pe._host.evict_blocks(L.addr_evict_blocks, desc, scores, t, n, budget, gone, freed) == pe.PE_OK
        else:
            pe.pe_score_triggered_blocks(desc, k, v, t, n, budget, scores)
            pe.pe_evict_blocks(desc, scores, t, n, budget, gone, freed)
        outs.append((t, n, scores, gone, freed))
    assert all(torch.equal(a, b) for a, b in zip(*outs)) and outs[0][1].tolist() == [16, 48, 32]
    with pytest.raises(ValueError, match="scores must be torch.float32"):
        pe.pe_evict_blocks(desc, outs[0][2].double(), *outs[0][:2], 48, *outs[0][3:])
    with pytest.raises(pe.PeError):   # no multiple of the page
        pe.pe_evict_blocks(desc, outs[0][2], *outs[0][:2], 40, *outs[0][3:])


CALLS = {"paged_decode", "append_paged_decode", "append_paged_decode_layers", "prefill_prune", "score_triggered_blocks",
         "score_recent_blocks", "evict_blocks", "evict_blocks_cached"}


class _Recorder:
    """The native marshalling, with a record of what each call returned."""

    def __init__(self, host):
        self.host, self.seen = host, []

    def __getattr__(self, name):
        def call(*args):
            status = getattr(self.host, name)(*args)
            self.seen.append((name, status))
            return status
        return call


def _engine_run(shared):
    """Prompts pruned and decode steps over two page boundaries, as engine.py makes the calls; every tensor that a call writes."""
    wl = synth.LLAMA32_1B.with_(dtype="f32", layers=2, num_kv_heads=Hk, num_q_heads=Hq, num_seqs=S, budget=64, steps=40)
    lens, written = [90, 64, 41], []

    def inputs(layers, step):
        per = [synth.decode_inputs(wl, l, step, 5, device="cuda") for l in range(layers)]
        return [torch.stack(t) for t in zip(*per)]

    for cached in (False, True):
        cache = PagedCache.create(torch.float32, S, Hk, Hq, D, B, synth.page_layout(wl, lens, 5, shared=shared), 64,
                                  shared=shared, decode_opts={"decode_splits": 2})
        cache.cached_scores = cached
        kept = torch.full((S, 64) if shared else (S, Hk, 64), -7, dtype=torch.int32, device="cuda")
        k, v, cu = synth.prompt_kv(wl, 0, lens, 5, device="cuda")
        cache.prefill_prune(k, v, cu, max(lens), kept)
        cache.set_host_lens(lens)
        cache.scores.fill_(float("inf"))
        for step in range(36):
            nk, nv, q = (t[0] for t in inputs(1, step))
            out = torch.empty_like(q)
            cache.decode_step(nk, nv, q, out, fused=step % 3 != 2)
            written.append(out)
        written += [kept, cache.block_table, cache.seq_lens, cache.k_pool, cache.v_pool, cache.scores, cache.freed_phys,
                    cache.evicted_logical, cache.spare_used]
    model = LayeredCache(torch.float32, 2, S, Hk, Hq, D, B, synth.page_layout(wl, lens * 2, 5, shared=shared), 64, shared=shared)
    for l in range(2):
        k, v, cu = synth.prompt_kv(wl, l, lens, 5, device="cuda")
        model.prefill_prune_layer(l, k, v, cu, max(lens))
    model.set_host_lens(lens)
    for step in range(36):
        nk, nv, q = inputs(2, step)
        out = torch.empty_like(q)
        model.decode_step(nk, nv, q, out)
        written.append(out)
    f = model.folded
    return written + [f.block_table, f.seq_lens, f.k_pool, f.v_pool, f.freed_phys, f.spare_used]


@pytest.mark.gpu
@pytest.mark.parametrize("shared", [False, True], ids=["per_head", "shared"])
def test_every_call_of_the_engine_goes_the_native_way_and_as_through_ctypes(monkeypatch, shared):
    pe.lib()
    recorder = _Recorder(pe._host)
    monkeypatch.setattr(pe, "_host", recorder)
    native = _engine_run(shared)
    assert {name for name, _ in recorder.seen} == CALLS and all(status == pe.PE_OK for _, status in recorder.seen)
    monkeypatch.setattr(pe, "_host", pe._NoHost())
    through_ctypes = _engine_run(shared)
    assert len(native) == len(through_ctypes) and all(torch.equal(a, b) for a, b in zip(native, through_ctypes))


@pytest.mark.gpu
def test_numbers_that_only_int_understands_go_through_ctypes(monkeypatch):
    """Budgets, lengths and counts as tensors of one element: taken before the native marshalling, and by the way through ctypes."""
    pe.lib()
    desc, q, k, v, table, lens = _args("cuda")
    lens = torch.tensor([16, 64, 48], dtype=torch.int32, device="cuda")
    i32 = dict(dtype=torch.int32, device="cuda")
    n = lambda x: torch.tensor(x)   # noqa: E731
    outs = []
    for wrap in (int, n):
        recorder = _Recorder(pe._host)
        with monkeypatch.context() as m:
            m.setattr(pe, "_host", recorder)
            t, sl, sl2, kp, vp = table.clone(), lens.clone(), torch.zeros(S, **i32), k.clone(), v.clone()
            scores = torch.zeros((S, Hk, PAGES), device="cuda")
            gone, freed, used = torch.full((S, Hk), -7, **i32), torch.full((S, Hk), -1, **i32), torch.zeros((S, Hk), **i32)
            pe.pe_score_recent_blocks(desc, kp, vp, t, sl, wrap(4), scores)
            pe.pe_evict_blocks_cached(desc, scores, t, sl, wrap(48), gone, freed)
            spare = torch.zeros((S, Hk, 1), **i32)
            new, out = torch.randn((S, Hk, D), generator=torch.Generator().manual_seed(1)).cuda(), torch.zeros_like(q)
            scale = 0.125 if wrap is int else n(0.125)
            one = sl.clone() - 1   # the tail pages have room
            pe.pe_append_paged_decode(desc, new, new, q, kp, vp, t, one, sl2, freed, spare, used, scale, out)
            out2 = torch.zeros_like(q)
            pe.pe_append_paged_decode_layers(desc, wrap(1), new, new, q, kp, vp, t, one, sl2, freed, spare, used, scale, out2)
            kp2, vp2, kept = torch.zeros_like(kp), torch.zeros_like(vp), torch.zeros((S, Hk, 32), **i32)
            tok = torch.randn((100, Hk, D), generator=torch.Generator().manual_seed(2)).cuda()
            cu = torch.tensor([0, 40, 80, 100], **i32)
            ws = pe.alloc_workspace(pe.PE_OP_PREFILL_PRUNE, desc, 100)
            pe.pe_prefill_prune(desc, tok, tok.flip(0), cu, wrap(100), wrap(40), wrap(32), kp2, vp2, table, sl2, kept, ws)
        assert [status for _, status in recorder.seen] == [pe.PE_OK if wrap is int else None] * 5
        outs.append([t, sl, sl2, kp, vp, scores, gone, freed, used, out, out2, kp2, vp2, kept])
    assert all(torch.equal(a, b) for a, b in zip(*outs))
