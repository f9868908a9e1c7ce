"""Which form of the attention kernel a descriptor leads to: the host layer of the library, built here with recording stand-ins for
the launches (no GPU needed)."""
import ctypes
import os
import subprocess

import pytest
import torch

from paper_2509_04377_amd import binding as pe
from paper_2509_04377_amd import build

STANDINS = r"""
#include "%s/pe_launch.h"
namespace pe {
static int seen[4];
hipError_t launch_score_blocks(const ScoreArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_score_evict(const ScoreEvictArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_evict_blocks(const EvictArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_append_kv(const AppendArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_prefill_prune(const PruneArgs&, hipStream_t) { return hipSuccess; }
size_t prune_workspace_bytes(int, int, int64_t, bool) { return 0; }
size_t decode_partials_bytes(int, int, int, int splits) { return splits > 1 ? 256 : 0; }
hipError_t launch_paged_decode(const DecodeArgs& a, hipStream_t) {
  seen[0] = a.splits;
  seen[1] = a.waves;
  seen[2] = a.depth;
  seen[3] = a.vector;
  return hipSuccess;
}
}  // namespace pe
extern "C" const int* seen_launch() { return pe::seen; }
"""


@pytest.fixture(scope="module")
def host_layer(tmp_path_factory):
    if torch.cuda.is_available() and torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the forms below are those of 256 compute units")
    d = tmp_path_factory.mktemp("routes")
    src, so = d / "standins.hip", d / "libroutes.so"
    src.write_text(STANDINS % build.CSRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.FLAGS + ["-O1", "-shared", str(src), os.path.join(build.CSRC, "pe_api.hip"), "-o", str(so)],
                   check=True, stderr=subprocess.DEVNULL)
    lib = ctypes.CDLL(str(so))
    lib.seen_launch.restype = ctypes.POINTER(ctypes.c_int)
    return lib


def _form(lib, **kw):
    """(splits, waves, tiles in flight) of pe_paged_decode for a descriptor."""
    d = dict(dtype=pe.PE_BF16, num_seqs=32, num_kv_heads=8, num_q_heads=32, head_dim=128, block_size=16, max_blocks=128,
             num_phys_blocks=4096)
    d.update(kw)
    desc, p = pe.make_desc(**d), ctypes.c_void_p(0x1000)   # the pointer goes to the stand-in only
    rc = lib.pe_paged_decode(ctypes.byref(desc), p, p, p, p, p, ctypes.c_float(0.1), p, p, ctypes.c_size_t(1 << 30), None)
    assert rc == pe.PE_OK
    return tuple(lib.seen_launch()[:3])


def _vector(lib, **kw):
    _form(lib, **kw)
    return bool(lib.seen_launch()[3])


def test_named_shapes_are_forms_of_their_own(host_layer):
    named = [_form(host_layer, decode_shape=s, decode_splits=1) for s in (424, 432, 822)]
    assert named == [(1, 4, 2), (1, 4, 3), (1, 8, 2)]
    for kw in (dict(), dict(num_seqs=4, max_blocks=256), dict(num_seqs=48)):
        assert _form(host_layer, decode_shape=422, **kw) == _form(host_layer, **kw)


@pytest.mark.parametrize("kw,want", [
    (dict(), (1, 8, 2)), (dict(max_blocks=127), (1, 4, 2)), (dict(head_dim=64, max_blocks=512), (1, 4, 2)),
    (dict(layout=pe.PE_LAYOUT_SHARED), (1, 4, 1)), (dict(num_seqs=31), (1, 4, 2)), (dict(num_seqs=48), (1, 4, 1)),
    (dict(num_seqs=48, head_dim=64), (1, 4, 1)), (dict(num_seqs=33), (4, 4, 1)), (dict(num_seqs=24, max_blocks=512), (4, 4, 1)),
    (dict(num_seqs=4, max_blocks=256), (8, 4, 1)), (dict(num_seqs=4, head_dim=64, max_blocks=256), (8, 4, 2)),
    (dict(num_seqs=1, max_blocks=100), (12, 4, 2)), (dict(max_blocks=4), (1, 4, 1)), (dict(num_seqs=4, max_blocks=4), (1, 4, 1)),
    (dict(num_seqs=4, max_blocks=5), (1, 4, 2)), (dict(num_seqs=16, decode_splits=2), (2, 4, 1)),
    (dict(num_seqs=8, decode_splits=2), (2, 4, 2))])
def test_bf16_form(host_layer, kw, want):
    assert _form(host_layer, **kw) == want


@pytest.mark.parametrize("kw,want", [
    (dict(head_dim=64, max_blocks=64), True), (dict(head_dim=64, max_blocks=65), False), (dict(max_blocks=12), True),
    (dict(max_blocks=13), False), (dict(num_seqs=33, head_dim=64, max_blocks=8), True), (dict(num_seqs=33, max_blocks=5), False),
    (dict(num_seqs=33, head_dim=64, max_blocks=9), False), (dict(num_seqs=33, max_blocks=4), True),
    (dict(num_q_heads=16, max_blocks=4), False), (dict(layout=pe.PE_LAYOUT_SHARED, max_blocks=4), False)])
def test_bf16_vector_units(host_layer, kw, want):
    assert _vector(host_layer, **dict(dict(num_q_heads=8), **kw)) is want


KERNEL = r"""
#include "%s/pe_decode_common.h"
__global__ void kernel(const int32_t* seq_lens, const int32_t* block_table, const void* q, const void* k_pool, const void* v_pool,
                       const int num_kv_heads, const int max_blocks, %s const uint32_t inv_heads, %s shape, const pe::DecodeParams) {}
hipError_t launch(const pe::DecodeKernelArgs& k) { return pe::launch_decode(kernel, dim3(1), dim3(64), nullptr, k); }
"""


@pytest.mark.parametrize("rows,max_blocks,want", [
    (64, 65, (4, 8, 1)), (80, 51, (3, 8, 1)), (40, 129, (6, 8, 1)), (32, 129, (8, 8, 1)), (20, 257, (12, 8, 1)), (8, 1025, (32, 8, 1)),
    (80, 35, (3, 4, 1)), (16, 129, (16, 4, 1)), (47, 257, (5, 8, 1)), (14, 257, (16, 8, 1))])
def test_bf16_eight_waves_by_one(host_layer, rows, max_blocks, want):
    """In eight splits and fewer, and in more, which are merged by a launch; not in pieces of fewer than 192 tokens."""
    assert _form(host_layer, num_seqs=rows, num_kv_heads=1, num_q_heads=8, max_blocks=max_blocks) == want


@pytest.mark.parametrize("kw,waves", [
    # whole rows: a table of 40 KiB with more than four query heads a KV head, of 48 KiB with fewer, and the next larger ones
    (dict(dtype=pe.PE_F32, num_q_heads=64, head_dim=64, max_blocks=5), 4), (dict(dtype=pe.PE_F32, num_q_heads=64, head_dim=64, max_blocks=6), 8),
    (dict(dtype=pe.PE_F32, head_dim=64, max_blocks=6), 4), (dict(dtype=pe.PE_F32, head_dim=64, max_blocks=7), 8),
    (dict(dtype=pe.PE_F32, max_blocks=3), 4), (dict(dtype=pe.PE_F32, max_blocks=4), 8), (dict(dtype=pe.PE_F32, num_seqs=1, max_blocks=1), 4),
    (dict(num_q_heads=8, max_blocks=6), 4), (dict(num_q_heads=8, max_blocks=7), 8),
    (dict(num_q_heads=8, head_dim=64, max_blocks=12), 4), (dict(num_q_heads=8, head_dim=64, max_blocks=13), 8),
    (dict(dtype=pe.PE_F32, num_seqs=33), 4), (dict(dtype=pe.PE_F32, num_seqs=8, max_blocks=64), 8), (dict(dtype=pe.PE_F32, num_seqs=32), 4),
    # split rows: eight wherever the workgroups are no more than the compute units
    (dict(num_seqs=1, num_q_heads=8, head_dim=64, max_blocks=57), 8), (dict(dtype=pe.PE_F32, num_seqs=1, head_dim=64, max_blocks=8, decode_splits=8), 8)])
def test_waves_on_the_vector_units(host_layer, kw, waves):
    assert _form(host_layer, **kw)[1] == waves


@pytest.mark.parametrize("more,last,compiles", [("", "const uint32_t", True), ("const int more,", "const uint32_t", False),
                                                ("", "const uint64_t", False)])
def test_attention_kernels_have_the_parameters_that_are_read_by_offset(tmp_path, more, last, compiles):
    """The kernels read their later arguments out of the argument segment; one with other parameters must not build."""
    src = tmp_path / "kernel.hip"
    src.write_text(KERNEL % (build.CSRC, more, last))
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    r = subprocess.run([hipcc] + build.FLAGS + ["--cuda-host-only", "-fsyntax-only", str(src)], stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True)
    assert (r.returncode == 0) == compiles, r.stdout
    assert compiles or "parameter of type 'DecodeKernel'" in r.stdout, r.stdout
