"""The native argument marshalling: what it takes, what it leaves to the way through ctypes (which accepts it or says what is
wrong), and that both make the same call."""
import ctypes

import pytest
import torch

from paper_2509_04377_amd import binding as pe

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
