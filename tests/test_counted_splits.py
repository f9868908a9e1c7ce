"""Splits that the last of them to arrive merges, counted (pe_append_paged_decode_layers from its second layer on) or tagged (single calls
and the first layer): which calls take which way, with the host layer built against recording stand-ins, and on the GPU the same steps in
either way and with a launch that merges the splits, as into an output that is not aligned to a tag."""
import ctypes
import math
import os
import subprocess

import pytest
import torch

from paper_2509_04377_amd import binding as pe
from paper_2509_04377_amd import build, synth
from paper_2509_04377_amd.engine import GraphedStepper, LayeredCache

STANDINS = r"""
#include "%s/pe_launch.h"
namespace pe {
static long long seen[64][3];
static unsigned long long tags[64];
static int launches;
hipError_t launch_score_blocks(const ScoreArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_score_evict(const ScoreEvictArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_evict_blocks(const EvictArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_append_kv(const AppendArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_prefill_prune(const PruneArgs&, hipStream_t) { return hipSuccess; }
size_t prune_workspace_bytes(int, int, int64_t, bool) { return 0; }
size_t decode_partials_bytes(int, int, int, int splits) { return splits > 1 ? 256 : 0; }
hipError_t launch_paged_decode(const DecodeArgs& a, hipStream_t) {
  seen[launches][0] = a.splits;
  seen[launches][1] = a.counted;
  tags[launches] = a.tagged ? a.tag : 0;
  seen[launches++][2] = (long long)a.next_out;
  return hipSuccess;
}
}  // namespace pe
extern "C" int count_launches() { return pe::launches; }
extern "C" void forget_launches() { pe::launches = 0; }
extern "C" const long long* seen_launches() { return &pe::seen[0][0]; }
extern "C" const unsigned long long* seen_tags() { return pe::tags; }
"""


@pytest.fixture(scope="module")
def host_layer(tmp_path_factory):
    if torch.cuda.is_available() and torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the counts below are those of 256 compute units")
    d = tmp_path_factory.mktemp("counted")
    src, so = d / "standins.hip", d / "libcounted.so"
    src.write_text(STANDINS % build.CSRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.FLAGS + ["-O1", "-shared", str(src), os.path.join(build.CSRC, "pe_api.hip"), "-o", str(so)],
                   check=True, stderr=subprocess.DEVNULL)
    lib = ctypes.CDLL(str(so))
    lib.seen_launches.restype = ctypes.POINTER(ctypes.c_longlong)
    lib.seen_tags.restype = ctypes.POINTER(ctypes.c_ulonglong)
    return lib


OUT, Q, NEW = 1 << 30, 1 << 34, 1 << 36


def _layers(lib, layers=3, out=OUT, q=Q, new=NEW, **kw):
    """[(splits, counted, next output)] of the attention launches of a call."""
    d = dict(dtype=pe.PE_BF16, num_seqs=8, num_kv_heads=8, num_q_heads=32, head_dim=64, block_size=16, max_blocks=65,
             num_phys_blocks=4096)
    d.update(kw)
    desc, p, v = pe.make_desc(**d), ctypes.c_void_p(1 << 40), ctypes.c_void_p
    lib.forget_launches()
    rc = lib.pe_append_paged_decode_layers(ctypes.byref(desc), layers, v(new), v(new + (1 << 32)), v(q), p, p, p, p, v(1 << 41), p, p, p, 2,
                                           ctypes.c_float(0.1), v(out), p, ctypes.c_size_t(1 << 30), None)
    assert rc == pe.PE_OK
    return [tuple(lib.seen_launches()[3 * i:3 * i + 3]) for i in range(lib.count_launches())], d


@pytest.mark.parametrize("kw,counted", [
    (dict(), True), (dict(dtype=pe.PE_F32), True), (dict(layout=pe.PE_LAYOUT_SHARED), True),
    (dict(layout=pe.PE_LAYOUT_SHARED, dtype=pe.PE_F32), False),             # two launches, the append before the attention
    (dict(max_blocks=31), False),                                          # whole rows
    (dict(decode_splits=2), True), (dict(num_seqs=2, decode_splits=12), True), (dict(num_seqs=2, decode_splits=13), False), (dict(num_seqs=4, decode_splits=9), False),
    (dict(num_seqs=4, num_q_heads=64, decode_splits=8), True), (dict(num_seqs=4, num_q_heads=64, decode_splits=9), False),
    (dict(num_q_heads=64), True), (dict(num_q_heads=64, head_dim=128), True), (dict(num_q_heads=40, head_dim=128), True),
    (dict(num_seqs=4, num_q_heads=64, head_dim=128, decode_splits=4), False), (dict(num_q_heads=64, head_dim=128, max_blocks=47), False),
    (dict(head_dim=128), True), (dict(num_seqs=16, decode_splits=4), True), (dict(num_seqs=17, decode_splits=4), False),
    (dict(head_dim=128, decode_shape=822), False), (dict(head_dim=128, decode_shape=432), False), (dict(head_dim=128, decode_shape=424), True)])
def test_which_calls_count(host_layer, kw, counted):
    seen, d = _layers(host_layer, **kw)
    bytes_ = d["num_seqs"] * d["num_q_heads"] * d["head_dim"] * (4 if d["dtype"] == pe.PE_F32 else 2)
    assert len(seen) == 3 and all(s[0] == seen[0][0] for s in seen)
    # the first layer's counts are cleared by nobody (it is tagged); every layer's are before its launch
    few = seen[0][0] <= 8   # (a launch merges nine to twelve, and clears the second layer's counts)
    assert [bool(t) for t in host_layer.seen_tags()[:3]] == [counted and few, False, False]
    assert [bool(s[1]) for s in seen] == [False, counted, counted]
    assert [s[2] for s in seen] == ([OUT + bytes_, OUT + 2 * bytes_, 0] if counted else [0, 0, 0])


@pytest.mark.parametrize("kw", [dict(layers=1), dict(out=OUT + 2), dict(out=OUT + 4), dict(q=OUT), dict(out=Q + 100), dict(new=OUT + 64), dict(new=OUT - (1 << 32))],
                         ids=["one layer", "odd address", "half a tag", "in place", "over q", "over new_k", "over new_v"])
def test_outputs_that_cannot_hold_counts(host_layer, kw):
    seen, _ = _layers(host_layer, **kw)
    assert seen == [(seen[0][0], 0, 0)] * kw.get("layers", 3) and seen[0][0] > 1
    assert [bool(t) for t in host_layer.seen_tags()[:len(seen)]] == [kw.get("layers") == 1] * len(seen)


@pytest.mark.parametrize("kw,out,q,tagged", [
    (dict(), OUT, Q, True), (dict(), OUT + 8, Q, True), (dict(), OUT + 4, Q, False), (dict(), Q, Q, False), (dict(), Q + 512, Q, False),
    (dict(dtype=pe.PE_F32), OUT, Q, True), (dict(dtype=pe.PE_F32, layout=pe.PE_LAYOUT_SHARED), OUT, Q, False),
    (dict(layout=pe.PE_LAYOUT_SHARED), OUT, Q, True), (dict(decode_splits=7), OUT, Q, True),
    (dict(num_seqs=4, decode_splits=8, max_blocks=511), OUT, Q, True), (dict(num_seqs=4, decode_splits=8, max_blocks=512), OUT, Q, False),
    (dict(num_seqs=4, decode_splits=9), OUT, Q, False), (dict(max_blocks=31), OUT, Q, False)])
def test_which_single_calls_tag(host_layer, kw, out, q, tagged):
    d = dict(dtype=pe.PE_BF16, num_seqs=8, num_kv_heads=8, num_q_heads=32, head_dim=64, block_size=16, max_blocks=65, num_phys_blocks=4096)
    d.update(kw)
    desc, p, v, ws = pe.make_desc(**d), ctypes.c_void_p(1 << 40), ctypes.c_void_p, ctypes.c_size_t(1 << 30)
    host_layer.forget_launches()
    for _ in range(2):
        assert host_layer.pe_append_paged_decode(ctypes.byref(desc), v(NEW), v(NEW + (1 << 32)), v(q), p, p, p, p, v(1 << 41), p, p, p, 2,
                                                 ctypes.c_float(0.1), v(out), p, ws, None) == pe.PE_OK
        assert host_layer.pe_paged_decode(ctypes.byref(desc), v(q), p, p, p, p, ctypes.c_float(0.1), v(out), p, ws, None) == pe.PE_OK
    tags = host_layer.seen_tags()[:4]
    assert [bool(t) for t in tags] == [tagged] * 4 and (not tagged or len(set(tags)) == 4)
    assert all(host_layer.seen_launches()[3 * i + 1] == host_layer.seen_launches()[3 * i + 2] == 0 for i in range(4))


def _engines(dtype, S, Hk, G, D, budget, B, shared, splits, n, layers=3):
    wl = synth.Workload("counted", 0, dtype, layers, Hk, G * Hk, D, B, S, (1,), budget, 2 * B, "lognormal", True)
    lens = [max(1, budget - 7 * s) for s in range(S)]
    out = []
    for _ in range(n):
        layout = synth.page_layout(wl, lens * layers, 3, shared=shared)
        e = LayeredCache(wl.torch_dtype, layers, S, Hk, G * Hk, D, B, layout, budget, "cuda", shared=shared,
                         decode_opts=dict(decode_splits=splits))
        g = torch.Generator(device="cuda")
        g.manual_seed(11)
        for pool in (e.folded.k_pool, e.folded.v_pool):
            pool.copy_(torch.randn(pool.shape, generator=g, device="cuda"))
        e.folded.seq_lens.copy_(torch.tensor(lens * layers, dtype=torch.int32, device="cuda"))
        e.set_host_lens(lens)
        out.append(e)
    return wl, out


def _inputs(wl, step):
    g = torch.Generator(device="cuda")
    g.manual_seed(100 + step)
    kv, qo = (wl.layers, wl.num_seqs, wl.num_kv_heads, wl.head_dim), (wl.layers, wl.num_seqs, wl.num_q_heads, wl.head_dim)
    return [torch.randn(s, generator=g, device="cuda").to(wl.torch_dtype) for s in (kv, kv, qo)]


def _same_state(a, b):
    for name in ("block_table", "seq_lens", "spare_used", "freed_phys", "k_pool", "v_pool"):
        x, y = getattr(a.folded, name), getattr(b.folded, name)
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name


SHAPES = [("bf16", 3, 2, 4, 64, 512, 16, False, 2), ("bf16", 3, 2, 3, 64, 1024, 16, False, 4), ("bf16", 2, 3, 8, 64, 2048, 32, False, 8),
          ("bf16", 2, 2, 1, 64, 512, 16, False, 5), ("bf16", 3, 8, 4, 128, 1024, 16, False, 7), ("bf16", 1, 1, 3, 128, 640, 64, False, 4),
          ("bf16", 2, 2, 4, 128, 64, 16, False, 12), ("bf16", 3, 3, 7, 64, 768, 16, True, 6), ("bf16", 2, 4, 2, 128, 512, 16, True, 3),
          ("bf16", 16, 8, 1, 128, 512, 16, False, 4), ("f32", 3, 2, 2, 64, 512, 16, False, 2), ("f32", 2, 3, 5, 64, 1024, 16, False, 7),
          ("f32", 2, 2, 3, 128, 512, 32, False, 4), ("f32", 1, 5, 1, 128, 2048, 16, False, 12), ("bf16", 1, 1, 2, 128, 512, 16, False, 15), ("bf16", 7, 8, 7, 128, 1024, 16, False, 4),
          ("bf16", 8, 8, 5, 128, 768, 32, True, 4), ("bf16", 3, 8, 8, 128, 2048, 16, False, 8), ("f32", 2, 8, 4, 128, 512, 16, False, 8)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,S,Hk,G,D,budget,B,shared,splits", SHAPES)
def test_counted_splits_equal_merged_ones(dtype, S, Hk, G, D, budget, B, shared, splits):
    """The same records, added up in another order: at most splits + 8 roundings to fp32 on either side, each of a sum that is no larger than
    the largest value, and for bf16 one rounding of the output on either side."""
    wl, (counted, again, merged, tagged) = _engines(dtype, S, Hk, G, D, budget, B, shared, splits, 4)
    merged.native_layers = tagged.native_layers = False
    shape = (wl.layers, S, wl.num_q_heads, D)
    odd = 4 // wl.torch_dtype.itemsize   # elements: an output that begins in the middle of a tag is merged by launches
    outs = [torch.full((math.prod(shape) + odd,), 7.0, device="cuda", dtype=wl.torch_dtype)[o:][:math.prod(shape)].view(shape)
            for o in (0, 0, odd, 0)]
    alone = [torch.empty_like(outs[0][0]), outs[2].new_empty(outs[2][0].numel() + odd)[odd:].view(shape[1:])]
    for step in range(B + 3):
        k, v, q = _inputs(wl, step)
        for e, o in zip((counted, again, merged, tagged), outs):
            e.decode_step(k, v, q, o)
        assert torch.equal(outs[0].view(torch.uint8), outs[1].view(torch.uint8)), "run to run, step %d" % step
        if splits < 8:
            assert torch.equal(outs[0].view(torch.uint8), outs[3].view(torch.uint8)), "counted and tagged, step %d" % step
        c = tagged.per_layer[step % wl.layers]   # the attention alone, over what was appended
        for o in alone:
            pe.pe_paged_decode(c.desc, q[step % wl.layers], c.k_pool, c.v_pool, c.block_table, c.seq_lens, D ** -0.5, o, c.decode_ws)
        largest = float(max(counted.folded.v_pool.abs().max(), v.abs().max()))
        for a, b in ((outs[0].double(), outs[2].double()), (alone[0].double(), alone[1].double())):
            tol = 2 * (splits + 8) * 2.0 ** -24 * largest + (2.0 ** -7 * b.abs() if dtype == "bf16" else 0.0)
            assert bool(((a - b).abs() <= tol).all()), (step, float((a - b).abs().max()))
    _same_state(counted, merged)
    _same_state(counted, tagged)


@pytest.mark.gpu
def test_counted_splits_in_place_of_the_queries():
    """An output that is the queries' own memory (no room for counts: the splits are merged by launches of their own)."""
    wl, (a, b) = _engines("bf16", 3, 2, 4, 64, 512, 16, False, 4, 2)
    for step in range(4):
        k, v, q = _inputs(wl, step)
        out, mine = torch.empty_like(q), q.clone()
        a.decode_step(k, v, q, out)
        b.decode_step(k, v, mine, mine)
        assert bool(((out.double() - mine.double()).abs() <= 2.0 ** -7 * out.double().abs() + 1e-4).all()), step
    _same_state(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,S,Hk,G,D,budget,B,shared,splits", [SHAPES[1], SHAPES[4], SHAPES[7], SHAPES[11]])
@pytest.mark.parametrize("native", [True, False], ids=["counted", "tagged"])
def test_counted_splits_from_a_graph(dtype, S, Hk, G, D, budget, B, shared, splits, native):
    """Replays, with eager work and synchronisations in between: every one clears the counts of the next launch itself, and leaves none of
    its tags, which a graph keeps, in the output."""
    wl, (eager, graphed) = _engines(dtype, S, Hk, G, D, budget, B, shared, splits, 2)
    graphed.native_layers = eager.native_layers = native
    k, v, q = _inputs(wl, 0)
    bufs = [x.clone() for x in (k, v, q)]
    out_g, out_e = torch.full_like(q, 3.0), torch.full_like(q, 5.0)
    stepper = GraphedStepper(graphed, *bufs, out_g)
    for step in range(2 * B + 3):
        for x, y in zip(bufs, _inputs(wl, step)):
            x.copy_(y)
        torch.cuda.synchronize()
        stepper.step()
        eager.decode_step(*bufs, out_e)
        torch.cuda.synchronize()
        assert torch.equal(out_g.view(torch.uint8), out_e.view(torch.uint8)), step
        out_g.fill_(float(step))   # what lies in the output between two steps does not matter
    _same_state(eager, graphed)


@pytest.mark.gpu
@pytest.mark.parametrize("splits", [2, 3, 5, 6, 7, 8, 11])
@pytest.mark.parametrize("D,G", [(64, 3), (128, 1)])
def test_an_infinity_stays_one(D, G, splits):
    """fp32, an infinite element in the first and in the last token of every row, so in the first and in the last split that is merged: these
    two elements of the results are infinite, as in a row that is not split, and every other one is what it is there (at most splits + 8 +
    len roundings of sums no larger than the largest value on either side, eight times the root of their number)."""
    shape, budget = ("f32", 2, 2, G, D, 640, 16, False), 640
    wl, (counted, merged, tagged) = _engines(*shape, splits, 3)
    _, (whole,) = _engines(*shape, 1, 1)
    merged.native_layers = tagged.native_layers = False
    k, v, q = _inputs(wl, 0)
    q = q * 0.1
    largest = float(max(whole.folded.v_pool.abs().max(), v.abs().max()))
    v[..., 3] = math.inf
    size = q.numel()
    outs = [torch.full((size + 1,), 7.0, device="cuda")[o:][:size].view(q.shape) for o in (0, 1, 0, 0)]
    for e, o in zip((counted, merged, tagged, whole), outs):
        e.folded.v_pool[e.folded.block_table[:, :, 0].long(), 0, 5] = -math.inf
        e.decode_step(k, v, q, o)
    want = outs[3]
    assert bool((want[..., 3] == math.inf).all()) and bool((want[..., 5] == -math.inf).all())
    finite = [d for d in range(D) if d not in (3, 5)]
    tol = 8 * (splits + 8 + budget) ** 0.5 * 2.0 ** -24 * largest
    for name, o in zip(("counted", "merged by a launch", "tagged"), outs):
        assert torch.equal(o[..., [3, 5]], want[..., [3, 5]]), name
        assert bool(((o - want)[..., finite].abs() <= tol).all()), name


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,S,Hk,G,D,budget,B,shared,splits", SHAPES + [
    ("f32", 2, 3, 5, 64, 1024, 16, False, 8), ("bf16", 2, 2, 4, 64, 1024, 16, False, 9), ("f32", 1, 2, 1, 64, 640, 16, False, 10)])
def test_every_way_gives_the_same_bits(dtype, S, Hk, G, D, budget, B, shared, splits):
    """Counted, tagged and merged by a launch (an output in the middle of a tag), layers in one call or one by one, the attention alone with
    a workspace and without: the splits are added in one order."""
    wl, engines = _engines(dtype, S, Hk, G, D, budget, B, shared, splits, 4)
    engines[2].native_layers = engines[3].native_layers = False
    odd = 4 // wl.torch_dtype.itemsize
    for step in range(3):
        k, v, q = _inputs(wl, step)
        size, outs = q.numel(), []
        for e, at in zip(engines, (0, odd, 0, odd)):
            out = torch.full((size + odd,), 7.0, device="cuda", dtype=wl.torch_dtype)[at:][:size].view(q.shape)
            e.decode_step(k, v, q, out)
            outs.append(out)
        for o in outs[1:]:
            assert torch.equal(outs[0], o)
        c, layer = engines[0].per_layer[step], q[step]
        alone = [torch.full((layer.numel() + odd,), 7.0, device="cuda", dtype=wl.torch_dtype)[at:][:layer.numel()].view(layer.shape)
                 for at in (0, odd, 0)]
        for o in alone[:2]:
            pe.pe_paged_decode(c.desc, layer, c.k_pool, c.v_pool, c.block_table, c.seq_lens, D ** -0.5, o, c.decode_ws)
        pe.pe_paged_decode_static(c.desc, layer, c.k_pool, c.v_pool, c.block_table, c.seq_lens, D ** -0.5, alone[2])
        assert torch.equal(alone[0], alone[1]) and torch.equal(alone[0], alone[2])
