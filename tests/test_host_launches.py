"""What the library's host code passes to its kernels, without a GPU: the
library's objects are linked with recording stand-ins for the HIP runtime
(launch_recorder.cpp), so every entry point runs to its launches.

Live-ray arrays (one byte and one mask per 64 rays, written by the traversal)
must lie inside the workspace that the caller was told to bring, for every
decoder shape that the size query accepts: also those that no kernel serves,
whose calls still traverse before they are refused, or only traverse."""

import ctypes as ct
import os
import subprocess

import pytest

from paper_2205_07058_amd import build, svlf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 1 << 40              # device addresses that nothing dereferences


@pytest.fixture(scope="module")
def rec(tmp_path_factory):
    objs = [os.path.join(build.BUILD, s + ".o") for s in build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        build.build()
    lib = str(tmp_path_factory.mktemp("rec") / "libsvlf_recorded.so")
    r = subprocess.run(["g++", "-O1", "-fPIC", "-std=c++17", "-shared", "-D__HIP_PLATFORM_AMD__", "-w", "-I",
                        "/opt/rocm/include", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, "-o", lib,
                        os.path.join(ROOT, "tests", "launch_recorder.cpp")] + objs +
                       ["-Wl,-Bsymbolic", "-Wl,-z,defs", "-lpthread"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    rec = ct.CDLL(lib)
    for name, (args, res) in svlf._SIGS.items():
        getattr(rec, name).argtypes, getattr(rec, name).restype = args, res
    rec.rec_live_begin.restype = rec.rec_live_end.restype = ct.c_uint64
    return rec


def _scene():
    sc = (svlf.Scene * 1)()
    o = sc[0].octree
    o.depth, o.n_leaves, o.n_vertices, o.n_nodes, o.nodes, o.leaf_corners = 5, 100, 300, 50, FAKE, FAKE
    sc[0].features = sc[0].features_bf16 = FAKE
    return sc


def _mlp(widths):
    m = svlf.Mlp()
    m.n_layers = len(widths) - 1
    m.widths[:len(widths)] = widths
    m.params = FAKE
    return m


def _render(rec, widths, n, K=8, flags=0):
    """Status of svlf_render of n rays in a workspace of exactly the size asked for, and that size."""
    m, opts, offs = _mlp(widths), svlf.make_opts(K, "voxel", "fp32", flags), (ct.c_int64 * 2)(0, n)
    size = rec.svlf_workspace_bytes(ct.byref(m), ct.byref(opts), n)
    assert size > 0
    rec.rec_reset()
    rc = rec.svlf_render(_scene(), 1, offs, ct.byref(m), ct.byref(opts), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, size,
                         None)
    return rc, size


@pytest.mark.parametrize("flags", [0, svlf.FLAG_TRACE_ONLY])
@pytest.mark.parametrize("n", [1 << 15, 1500001, 1 << 22])
@pytest.mark.parametrize("widths", [(8, 32, 4), (16, 32, 4), (8, 32, 32, 4), (16, 64, 64, 64, 4), (32, 64, 64, 64, 4)])
def test_live_arrays_inside_the_workspace(rec, widths, n, flags):
    rc, size = _render(rec, widths, n, flags=flags)
    served = widths in ((8, 32, 32, 4), (16, 64, 64, 64, 4), (32, 64, 64, 64, 4))
    assert rc == (svlf.OK if served or flags else svlf.E_UNSUPPORTED)
    assert rec.rec_traces() == 1
    assert rec.rec_live_traces() == 1 or not served
    if rec.rec_live_traces():
        assert FAKE <= rec.rec_live_begin() and rec.rec_live_end() <= FAKE + size


def _lf_model():
    m = svlf.LfModel()
    m.c_density, m.c_color, m.hidden, m.n_hidden_density, m.n_hidden_color = svlf.LF_DECODERS
    m.params = FAKE
    return m


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("K", [1, 8, 16])
@pytest.mark.parametrize("call", ["render", "lf_render", "lf"])
def test_workspace_size_grows_with_the_rays(rec, call, K, precision):
    """A workspace sized for some rays serves every call with fewer."""
    opts = svlf.make_opts(K, "voxel", precision)
    m, query = (_mlp((8, 32, 32, 4)), rec.svlf_workspace_bytes) if call == "render" else (
        _lf_model(), getattr(rec, f"svlf_{call}_workspace_bytes"))
    edges = [1, 64, 4096, 1 << 15, 1 << 18, 1 << 20, 1 << 22, (1 << 22) + 1345, (1 << 22) + 9857, 1 << 23]
    ns = sorted({e + k for e in edges for k in (-64, -1, 0, 1, 63, 64) if e + k > 0})
    sizes = [query(ct.byref(m), ct.byref(opts), n) for n in ns]
    assert all(0 < a <= b for a, b in zip(sizes, sizes[1:])), [n for n, a, b in zip(ns, sizes, sizes[1:]) if a > b]


@pytest.mark.parametrize("n", [40009, 1 << 18])
def test_lf_render_makes_no_live_arrays(rec, n):
    """The light field's forward kernels take items over all rays: a render neither asks for room for the
    live-ray arrays nor has the traversal write them; a backward pass does both."""
    m, opts, offs = _lf_model(), svlf.make_opts(4, "direct", "fp32"), (ct.c_int64 * 2)(0, n)
    args = (_scene(), 1, offs, ct.byref(m), ct.byref(opts), FAKE, FAKE)
    size = rec.svlf_lf_render_workspace_bytes(ct.byref(m), ct.byref(opts), n)
    rec.rec_reset()
    assert rec.svlf_lf_render(*args, FAKE, FAKE, FAKE, FAKE, size, None) == svlf.OK
    assert (rec.rec_traces(), rec.rec_live_traces()) == (1, 0)
    full = rec.svlf_lf_workspace_bytes(ct.byref(m), ct.byref(opts), n)
    assert full - size >= (n + 63) // 64 * 9
    rec.rec_reset()
    assert rec.svlf_lf_render_backward(*args, FAKE, FAKE, FAKE, (ct.c_void_p * 1)(FAKE), FAKE, FAKE, full, None) == svlf.OK
    assert (rec.rec_traces(), rec.rec_live_traces()) == (1, 1)
    assert FAKE <= rec.rec_live_begin() and rec.rec_live_end() <= FAKE + full


def test_lds_limit_does_not_depend_on_the_call(rec):
    """A kernel's dynamic-LDS limit is state of the process: threads that launch the same kernel with different K
    must not set it to different values between each other's set and launch."""
    rec.rec_reset()
    for widths in ((8, 32, 32, 4), (16, 64, 64, 64, 4), (32, 64, 64, 64, 4)):
        for K in (16, 1, 9):
            assert _render(rec, widths, 4096, K=K)[0] == svlf.OK
            assert rec.rec_lds_limit_changes() == 0, (widths, K)


def test_first_round_of_items_is_dealt(rec):
    """Blocks start on items of their own: the counter that hands out the last two rounds would serve all blocks of
    the first round one after the other."""
    for blocks in (1, 7, 256, 896):
        for n in (0, 1, blocks - 1, blocks, blocks + 1, 2 * blocks, 3 * blocks - 1, 3 * blocks, 3 * blocks + 1,
                  20 * blocks + 3):
            dealt = rec.rec_dealt_items(n, blocks)
            assert min(n, blocks) <= dealt <= n and n - dealt <= 2 * blocks
            assert n < 3 * blocks or dealt == n - 2 * blocks


@pytest.mark.parametrize("n,live", [((1 << 15) - 1, 0), (1 << 15, 1), (262145, 1), (1 << 22, 1), ((1 << 22) + 1, 0)])
def test_reused_hits_get_the_live_plan(rec, n, live):
    """A call that reuses hits has its items planned like one that traverses: the live-ray arrays are made from the
    counts, inside the workspace."""
    rc, size = _render(rec, (8, 32, 32, 4), n, flags=svlf.FLAG_REUSE_HITS)
    assert rc == svlf.OK and rec.rec_traces() == 0 and rec.rec_live_counts() == live and rec.rec_launches() == 2
    if live:
        assert FAKE <= rec.rec_live_begin() and rec.rec_live_end() <= FAKE + size
    # no room (a decoder that no kernel serves): over all rays
    assert _render(rec, (8, 32, 4), n, flags=svlf.FLAG_REUSE_HITS)[0] == svlf.E_UNSUPPORTED
    assert rec.rec_live_counts() == (live and n < 1 << 20)
