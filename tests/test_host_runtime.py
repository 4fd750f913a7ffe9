"""Decisions of the library's host code -- what is allocated when, what is
launched -- against a HIP runtime that runs nothing (host_hip_stub.c), without
a GPU.  Each test is a program of its own, in a process of its own."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

from paper_2405_14105_amd import dsi

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("gcc") is None or not os.path.exists(dsi.LIB_PATH),
                                reason="needs gcc and the built library")

PRELUDE = '''
import ctypes, re, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
hip.stub_budget.argtypes = [ctypes.c_size_t]
hip.stub_in_use.restype = ctypes.c_size_t
hip.stub_log.restype = hip.stub_kernel.restype = ctypes.c_char_p
import dsi_synth as S
from paper_2405_14105_amd import dsi
STREAM, P = 1, 4096                     # any addresses: nothing reads them

def model(shape, layers=None):
    kind = {"bf16": dsi.DSI_BF16, "f32": dsi.DSI_F32}
    L = layers or shape.n_layers
    m = dsi.dsi_model_create(dsi.make_config(L, shape.d_model, shape.n_heads, shape.n_kv_heads, shape.head_dim, shape.d_ff,
                             shape.vocab, wdtype=kind[shape.wdtype], kvdtype=kind[shape.kvdtype]), STREAM)
    e = 4 if shape.wdtype == "f32" else 2
    for l in range(-1, L):
        for name in (S.GLOBAL_TENSORS if l < 0 else S.LAYER_TENSORS):
            n = 1
            for x in S.tensor_shape(shape, name):
                n *= x
            dsi.dsi_model_set_tensor(m, l, dsi.TENSOR_IDS[name], P, n * e, True)
    hip.stub_clear()
    return m

def kernel(name):
    """(kernel, its template arguments)"""
    k = re.search(r"\\d(k_[a-z0-9_]+)", name)
    assert k, name
    return k[1], tuple(int(v) for v in re.findall(r"L[ij](\\d+)E", name))

def launches():
    """(kernel, its template arguments, grid) of the launches since the last stub_clear()."""
    out = []
    for line in hip.stub_log().decode().splitlines():
        name, x, y, z, b = line.rsplit(" ", 4)
        out.append(kernel(name) + ((int(x), int(y), int(z)),))
    return out

def built():
    return {kernel(hip.stub_kernel(i).decode()) for i in range(hip.stub_kernels())}
'''


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip") / "libstub.so")
    r = subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "host_hip_stub.c"), "-o", so],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return so


def run(stub, program):
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(program), stub], capture_output=True, text=True,
                       env=env, cwd=ROOT, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]


def test_short_forwards_can_be_captured_after_a_long_prompt(stub):
    """A long prompt leaves the buffers that captured short prompts and drafts on the same cache need."""
    run(stub, '''
    for name in ("gqa_hd64", "tiny", "mha_hd128"):
        for n in (65, 100, 130, 900):
            m = model(S.SHAPES[name])
            kv = dsi.dsi_kv_create(m, 1, 4000)
            dsi.dsi_prefill(m, kv, 0, P, n, P)
            dsi.dsi_kv_rollback(kv, 0, n - 64)
            hip.stub_capture(1)
            dsi.dsi_prefill(m, kv, 0, P, 40, P)
            dsi.dsi_kv_rollback(kv, 0, n - 64)
            dsi.dsi_draft(m, kv, 0, P, 2, 5, P, P, P)
            hip.stub_capture(0)
            assert hip.stub_refused() == 0
            dsi.dsi_kv_destroy(kv)
            dsi.dsi_model_destroy(m)
    ''')


def test_growing_buffers_free_nothing(stub):
    """Buffers that captured launches may use are kept when longer calls need larger ones, and all are freed with the model."""
    run(stub, '''
    m = model(S.SHAPES["many_kv"])
    kv = dsi.dsi_kv_create(m, 4, 30000)
    hip.stub_clear()
    sizes = []
    for n in (10, 40, 64, 65, 300, 2000, 5000, 9000, 13000):
        dsi.dsi_prefill(m, kv, 0, P, n, P)
        sizes.append(hip.stub_mallocs())
    dsi.dsi_verify(m, kv, 0, 4, 5, P, P, P, P, P)
    assert hip.stub_frees() == 0
    assert hip.stub_mallocs() <= 12                    # sizes double
    dsi.dsi_kv_destroy(kv)
    dsi.dsi_model_destroy(m)
    assert hip.stub_in_use() == 0
    ''')


def test_prompt_workspace_under_memory_pressure(stub):
    """Where the whole workspace does not fit, a smaller one is taken; a refusal ends with the shortage."""
    run(stub, '''
    shape = S.SHAPES["llama1b"]
    def forwards(n=2000):
        hip.stub_clear()
        dsi.dsi_prefill(m, kv, 0, P, n, P)
        dsi.dsi_kv_rollback(kv, 0, 0)
        return sum(k == "k_prefill_rows" for k, _, _ in launches())    # of wide forwards; 0: 64-row ones
    m = model(shape, layers=1)
    kv, other = (dsi.dsi_kv_create(m, 1, 2048) for _ in range(2))
    dsi.dsi_prefill(m, other, 0, P, 10, P)
    dsi.dsi_prefill(m, kv, 0, P, 64, P)                 # the 64-row forwards' buffers
    dsi.dsi_kv_rollback(kv, 0, 0)
    base = hip.stub_in_use()
    assert forwards() == 1
    whole = hip.stub_in_use() - base
    m = model(shape, layers=1)
    kv = dsi.dsi_kv_create(m, 1, 2048)
    other = dsi.dsi_kv_create(m, 1, 2048)
    hip.stub_budget(whole * 3 // 4)
    assert forwards() == 2                              # half the rows
    hip.stub_budget(1 << 40)
    counts = [forwards() for _ in range(20)]
    assert counts[0] == 2 and counts[-1] == 1           # the whole, some prompts later
    m = model(shape, layers=1)
    kv = dsi.dsi_kv_create(m, 1, 2048)
    other = dsi.dsi_kv_create(m, 1, 2048)
    hip.stub_budget(32 << 20)
    assert forwards() == 0
    hip.stub_budget(1 << 40)
    assert forwards() == 0
    dsi.dsi_kv_destroy(other)                           # memory came back
    assert forwards() == 1
    ''')


def test_prompt_cases_launch_every_variant(stub):
    """Every variant of the prefill GEMM that is built is one that a prompt of wide_cases.py launches."""
    run(stub, '''
    sys.path.insert(0, "tests")
    from wide_cases import WIDE_CASES
    seen = set()
    for d, hq, hkv, hd, ff, n in WIDE_CASES:
        m = model(S.Shape("case", 2, d, hq, hkv, hd, ff, 256, kvdtype="f32"))
        kv = dsi.dsi_kv_create(m, 2, 21 + n)
        dsi.dsi_prefill(m, kv, 0, P, n, P)
        here = {l[:2] for l in launches() if l[0] in ("k_gemm_wide", "k_wide_fold")}
        assert here, (d, ff, n)
        seen |= here
        dsi.dsi_kv_destroy(kv)
        dsi.dsi_model_destroy(m)
    want = {k for k in built() if k[0] in ("k_gemm_wide", "k_wide_fold")}
    assert len(want) > 20 and seen == want, (sorted(want - seen), sorted(seen - want))
    ''')


def test_weight_copies_give_way(stub):
    """A model and a cache that fit without the second copy of the weights are not refused for it."""
    run(stub, '''
    shape = S.SHAPES["llama13b"]
    GB = 1 << 30
    def rings(kv, rows=11):
        hip.stub_clear()
        dsi.dsi_verify(m, kv, 0, 1, rows - 1, P, P, P, P, P, commit=False)
        n = [k for k, _, _ in launches()]
        return sum(k == "k_gemm_ring" for k in n), sum(k == "k_gemm_bf16" for k in n)
    # room for everything
    m = model(shape, 4)
    used = hip.stub_in_use()
    kv = dsi.dsi_kv_create(m, 1, 32768)
    cache = hip.stub_in_use() - used
    assert rings(kv) == (17, 0)
    dsi.dsi_kv_destroy(kv)
    dsi.dsi_model_destroy(m)
    assert hip.stub_in_use() == 0
    # the model alone has no room for the copies
    hip.stub_budget(used * 6 // 10)
    m = model(shape, 4)
    hip.stub_budget(cache + (1 << 28))
    kv = dsi.dsi_kv_create(m, 1, 32768)
    assert rings(kv) == (0, 17)
    dsi.dsi_kv_destroy(kv)
    dsi.dsi_model_destroy(m)
    assert hip.stub_in_use() == 0
    # a cache comes later and needs their room; calls go on, in graphs of the library's too
    for late in (False, True):
        hip.stub_budget(used + 2 * cache)
        m = model(shape, 4)
        a = dsi.dsi_kv_create(m, 1, 32768)
        if late:
            assert rings(a) == (17, 0)
            dsi.dsi_prefill(m, a, 0, P, 300, P)
        hip.stub_budget(cache)
        b = dsi.dsi_kv_create(m, 1, 32768 + 4096)
        assert rings(a) == (0, 17) and rings(b) == (0, 17)
        dsi.dsi_prefill(m, b, 0, P, 300, P)
        dsi.dsi_kv_destroy(a)
        dsi.dsi_kv_destroy(b)
        dsi.dsi_model_destroy(m)
        assert hip.stub_in_use() == 0
    # a cache that would not fit without them either takes nothing
    hip.stub_budget(used + 2 * cache)
    m = model(shape, 4)
    a = dsi.dsi_kv_create(m, 1, 32768)
    dsi.dsi_prefill(m, a, 0, P, 300, P)
    hip.stub_budget(cache)
    before = hip.stub_in_use()
    try:
        dsi.dsi_kv_create(m, 4, 32768)
    except dsi.DsiError as e:
        assert e.status == dsi.DSI_ENOMEM
    else:
        raise AssertionError("a cache larger than the memory")
    assert hip.stub_in_use() == before and rings(a) == (17, 0)
    dsi.dsi_kv_destroy(a)
    dsi.dsi_model_destroy(m)
    # a graph of the caller's may hold them: then they stay
    hip.stub_budget(used + 2 * cache)
    m = model(shape, 4)
    a = dsi.dsi_kv_create(m, 1, 32768)
    dsi.dsi_prefill(m, a, 0, P, 60, P)
    hip.stub_capture(1)
    dsi.dsi_prefill(m, a, 0, P, 60, P)
    hip.stub_capture(0)
    hip.stub_budget(cache)
    hip.stub_clear()
    try:
        dsi.dsi_kv_create(m, 1, 32768 + 4096)
    except dsi.DsiError as e:
        assert e.status == dsi.DSI_ENOMEM
    else:
        raise AssertionError("a cache larger than the memory")
    assert hip.stub_frees() <= 2 and rings(a) == (17, 0)     # of the failed attempt
    ''')
