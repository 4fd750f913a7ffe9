"""Prompts longer than one 64-row chunk (many chunks in one forward) against
the fp64 oracle and against the same prompt in 64-token calls."""
import numpy as np
import pytest

import dsi_synth as S
from oracle import forward64
from oracle.model import embed64, layer64
from paper_2405_14105_amd import dsi
from parity import reg_of
from wide_cases import WIDE_CASES

pytestmark = pytest.mark.gpu
SEED = 5


def _rig(*a):
    from gpu_rig import Rig
    return Rig(*a)


def _weights(shape):
    return lambda l, n: S.weight(shape, SEED, l, n).astype(np.float64)


# one row past a chunk, one row past a tile, two and three row tiles of four and
# five blocks (every GEMM variant: test_every_gemm_variant); prefixes that end
# off the 16-, 32- and 64-row grids; group sizes 1, 3, 4 and 16; ragged FFN, K
# splits of O and down; several key chunks
@pytest.mark.parametrize("name,prefix,n", [
    ("ragged_bf16", 0, 65), ("ragged_bf16", 5, 129), ("gqa_hd64", 0, 97), ("gqa_hd64", 37, 257),
    ("mha_hd128", 63, 112), ("mha_hd128", 700, 66), ("many_kv", 0, 200), ("o_ring_hd128", 64, 300),
    ("ring_wide_ff", 31, 81), ("ring_wide_d", 0, 70),
    # fp32 weights and / or cache
    ("tiny", 0, 65), ("tiny", 40, 300), ("tiny", 33, 49), ("tiny", 9, 64), ("ragged_f32", 7, 130), ("hd96_kvf32", 33, 129), ("f32w_bf16kv", 0, 200)])
def test_matches_oracle(name, prefix, n):
    shape = S.SHAPES[name]
    toks = S.prefix_tokens(shape, SEED, 0, prefix + n)
    with _rig(shape, SEED, 2, prefix + n + 3) as rig:
        if prefix:
            rig.prefill(1, toks[:prefix])
        z = rig.prefill(1, toks[prefix:], want_logits=True)
        assert rig.length(1) == prefix + n
        kv = [rig.export_kv(1, l, prefix + n) for l in range(shape.n_layers)]
    zo, cache = forward64(shape, _weights(shape), toks)
    err = float(np.abs(z - zo[-1]).max())
    print(f"{name} {prefix}+{n}: max|dz| = {err:.3g}")
    assert err <= reg_of(shape)
    # keys and values: one bf16 spacing of the row's largest entry, or the
    # activations' own error (bf16 hi + lo, or fp32) in an fp32 cache
    rel = 2.0 ** -7 if shape.kvdtype == "bf16" else 1e-4 if shape.wdtype == "bf16" else 1e-5
    for l, (k, v) in enumerate(kv):
        for got, want in ((k, cache[l][0]), (v, cache[l][1])):
            want = np.asarray(want).reshape(got.shape)
            top = np.abs(want).max(axis=-1, keepdims=True)
            assert np.all(np.abs(got - want) <= rel * top + 1e-6)


# the limits are about half of what one running sum costs: over a wave's 64
# k-blocks of 4096 features, 0.9 % more error than in eight waves' runs of 16;
# over all keys of a row, 5-9 % more than in waves that take 32 keys each
@pytest.mark.parametrize("name,prefix,n,limit", [("wide_sums", 0, 700, 1.0045), ("tiny", 50, 300, 1.03),
                                                 ("tiny", 1000, 300, 1.03)])
def test_sums_are_no_less_exact_than_in_32_token_calls(name, prefix, n, limit):
    """Keys and values of the last layer in an fp32 cache, against fp64: a long prompt's error and 32-token calls'.
    The prefix's keys and values are of unit scale, so that attention is a good part of the residual."""
    import torch
    shape = S.SHAPES[name]
    toks = S.prefix_tokens(shape, SEED, 0, n)
    rng = np.random.default_rng(prefix)
    past = [[rng.standard_normal((prefix, shape.n_kv_heads, shape.head_dim)).astype(np.float32) for _ in range(2)]
            for _ in range(shape.n_layers)]
    last = shape.n_layers - 1
    with _rig(shape, SEED, 2, prefix + n) as rig:
        for w in (0, 1):
            for l in range(shape.n_layers if prefix else 0):
                kv = [torch.from_numpy(np.ascontiguousarray(x.transpose(1, 0, 2))).cuda() for x in past[l]]
                dsi.dsi_kv_import(rig.kv, w, l, prefix, *kv)
                torch.cuda.synchronize()
            dsi.dsi_kv_set_length(rig.kv, w, prefix)
        rig.prefill(0, toks)
        for i in range(0, n, 32):
            rig.prefill(1, toks[i:i + 32])
        wide, narrow = rig.export_kv(0, last, prefix + n), rig.export_kv(1, last, prefix + n)
    get = _weights(shape)
    x, pos = embed64(get, toks), prefix + np.arange(n)
    for l in range(shape.n_layers):
        x, k, v = layer64(shape, get, l, x, pos, *past[l])
    for a, b, want in zip(wide, narrow, (k, v)):
        ea, eb = (float(np.linalg.norm(y[prefix:] - want) / np.linalg.norm(want)) for y in (a, b))
        print(f"{name} {prefix}+{n}: {ea:.4g} against {eb:.4g}, {ea / eb:.4f}")
        assert ea <= limit * eb


@pytest.mark.parametrize("d,hq,hkv,hd,ff,n", WIDE_CASES)
def test_every_gemm_variant(d, hq, hkv, hd, ff, n):
    """Every tile, split, epilogue and fold of the prefill GEMM, against the window kernels (calls of at most 32 rows, which
    other tests hold to the oracle): last row's logits, keys and values of both layers, in an fp32 cache.  The bound is the
    one of test_matches_oracle for bf16 hi + lo activations."""
    import torch
    V, prefix = 256, 21
    g = torch.Generator(device="cuda").manual_seed(n)
    m = dsi.dsi_model_create(dsi.make_config(2, d, hq, hkv, hd, ff, V, kvdtype=dsi.DSI_F32), torch.cuda.current_stream().cuda_stream)
    kv = None
    try:
        def put(layer, name, *shape):
            w = torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16).mul_(0.02)
            if name.endswith("norm"):
                w.mul_(5).add_(1)
            torch.cuda.synchronize()
            dsi.dsi_model_set_tensor(m, layer, dsi.TENSOR_IDS[name], w.data_ptr(), w.numel() * 2, True)
        put(-1, "embed", V, d), put(-1, "final_norm", d), put(-1, "lm_head", V, d)
        for l in range(2):
            put(l, "attn_norm", d), put(l, "ffn_norm", d)
            put(l, "wq", hq * hd, d), put(l, "wk", hkv * hd, d), put(l, "wv", hkv * hd, d), put(l, "wo", d, hq * hd)
            put(l, "w_gate", ff, d), put(l, "w_up", ff, d), put(l, "w_down", d, ff)
        kv = dsi.dsi_kv_create(m, 2, prefix + n)
        toks = torch.randint(0, V, (prefix + n,), generator=g, device="cuda", dtype=torch.int32)
        z = torch.full((2, V), float("nan"), device="cuda")
        dsi.dsi_prefill(m, kv, 0, toks, prefix)
        dsi.dsi_prefill(m, kv, 0, toks[prefix:], n, z[0])
        for i in range(0, prefix + n, 32):
            dsi.dsi_prefill(m, kv, 1, toks[i:], min(32, prefix + n - i), z[1])
        out = [[torch.full((hkv, prefix + n, hd), float("nan"), device="cuda") for _ in range(4)] for _ in range(2)]
        for w in range(2):
            for l in range(2):
                dsi.dsi_kv_export(kv, w, l, prefix + n, out[w][2 * l], out[w][2 * l + 1])
        assert dsi.dsi_kv_length(kv, 0) == dsi.dsi_kv_length(kv, 1) == prefix + n
        worst = [float(((a - b).abs() / b.abs().amax(-1, keepdim=True)).max()) for a, b in zip(*out)]
        dz = float((z[0] - z[1]).abs().max() / z[1].abs().max())
        print(f"{(d, hq, hkv, hd, ff, n)}: {dz:.2g}, keys and values {max(worst):.2g}")
        assert dz <= 1e-4 and max(worst) <= 1e-4
    finally:
        torch.cuda.synchronize()
        if kv:
            dsi.dsi_kv_destroy(kv)
        dsi.dsi_model_destroy(m)


def test_more_than_one_forward():
    """2100 rows: two forwards; the rows of the second attend to the first's."""
    shape = S.SHAPES["gqa_hd64"]
    toks = S.prefix_tokens(shape, SEED, 0, 2100)
    with _rig(shape, SEED, 2, 2200) as rig:
        z = rig.prefill(0, toks, want_logits=True)
        for i in range(0, 2100, 64):        # one chunk a call
            z64 = rig.prefill(1, toks[i:i + 64], want_logits=True)
        assert rig.length(0) == rig.length(1) == 2100
    assert np.abs(z - z64).max() <= 2e-3


@pytest.mark.parametrize("bad", [(70,), (0, 199), (10, 140), (64, 70, 130, 210)])
@pytest.mark.parametrize("name", ["gqa_hd64", "tiny"])
def test_invalid_ids_drop_their_chunks(name, bad):
    """A chunk of 64 with an id outside the vocabulary is not cached, the others are, as in 64-token calls."""
    shape = S.SHAPES[name]
    n = 211
    toks = np.array(S.prefix_tokens(shape, SEED, 0, n))
    for i in bad:
        toks[i] = shape.vocab if i % 2 else -1
    with _rig(shape, SEED, 2, 300) as rig:
        rig.prefill(0, toks)
        for i in range(0, n, 64):
            rig.prefill(1, toks[i:i + 64])
        lens = []
        for w in (0, 1):
            try:
                rig.length(w)
                seen = False
            except dsi.DsiError as e:
                seen = e.status == dsi.DSI_EINVAL
            assert seen == (w == 0)          # one report for both windows' prompts
            lens.append(rig.length(w))
        chunks = {i // 64 for i in bad}
        assert lens[0] == lens[1] == sum(min(64, n - 64 * c) for c in range(4) if c not in chunks)
        for l in range(shape.n_layers):
            for a, b in zip(rig.export_kv(0, l, lens[0]), rig.export_kv(1, l, lens[0])):
                assert np.all(np.abs(a - b) <= 2.0 ** -7 * np.abs(b).max(axis=-1, keepdims=True) + 1e-6)


@pytest.mark.parametrize("name", ["mha_hd128", "tiny"])
def test_dead_rows_do_not_reach_the_logits(name):
    """Rows past the length hold NaN: a long prompt over them is not touched by it."""
    shape = S.SHAPES[name]
    toks = S.prefix_tokens(shape, SEED, 0, 150)
    with _rig(shape, SEED, 1, 400) as rig:
        a = rig.prefill(0, toks, want_logits=True)
        dsi.dsi_kv_rollback(rig.kv, 0, 0)
        dsi.dsi_kv_poison(rig.kv, 0)
        b = rig.prefill(0, toks, want_logits=True)
    assert np.all(np.isfinite(b)) and np.array_equal(a, b)


@pytest.mark.parametrize("name", ["gqa_hd64", "hd96_kvf32", "tiny"])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 100])
@pytest.mark.parametrize("off", [0, 1])
def test_cache_import_export_round_trip(name, n, off):
    """Every element comes back, from buffers at any element offset, and the rows past the imported ones stay."""
    import torch
    shape = S.SHAPES[name]
    dt = torch.bfloat16 if shape.kvdtype == "bf16" else torch.float32
    size = shape.n_kv_heads * n * shape.head_dim

    def buf():
        t = torch.randn(size + 8, device="cuda").to(dt)
        return t, t.data_ptr() + off * t.element_size()

    with _rig(shape, SEED, 2, 128) as rig:
        whole = [torch.randn((shape.n_kv_heads, 128, shape.head_dim), device="cuda").to(dt) for _ in range(2)]
        (k, kp), (v, vp) = buf(), buf()
        l = shape.n_layers - 1
        dsi.dsi_kv_import(rig.kv, 1, l, 128, *whole)
        dsi.dsi_kv_import(rig.kv, 1, l, n, kp, vp)
        (k2, k2p), (v2, v2p) = buf(), buf()
        dsi.dsi_kv_export(rig.kv, 1, l, n, k2p, v2p)
        got = [torch.empty_like(t) for t in whole]
        dsi.dsi_kv_export(rig.kv, 1, l, 128, *got)
        torch.cuda.synchronize()
        for a, b, full, back in ((k, k2, whole[0], got[0]), (v, v2, whole[1], got[1])):
            assert torch.equal(a[off:off + size], b[off:off + size])
            assert torch.equal(back[:, :n].reshape(-1), a[off:off + size]) and torch.equal(back[:, n:], full[:, n:])


def test_captured_prompt():
    """A prompt captured before any ran on the model (64-row forwards) and one captured after (wide), replayed."""
    import torch
    from gpu_rig import Rig
    shape = S.SHAPES["gqa_hd64"]
    toks = S.prefix_tokens(shape, SEED, 0, 150)
    with torch.cuda.stream(torch.cuda.Stream()), Rig(shape, SEED, 2, 200) as rig:
        t = rig.dev_i32(toks)
        rig.prefill(1, toks[:64])                    # the 64-row forwards' buffers
        out = []
        for after in (False, True):
            z = torch.zeros(shape.vocab, device="cuda")
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
                dsi.dsi_kv_rollback(rig.kv, 0, 0)
                dsi.dsi_prefill(rig.model, rig.kv, 0, t, len(toks), z)
            for _ in range(3):
                z.zero_()
                g.replay()
                torch.cuda.synchronize()
                out.append(z.cpu().numpy())
            dsi.dsi_kv_rollback(rig.kv, 0, 0)
            out.append(rig.prefill(0, toks, want_logits=True))
            dsi.dsi_kv_rollback(rig.kv, 0, 0)
    narrow, wide = out[0], out[3]
    assert all(np.array_equal(x, narrow) for x in out[:3]) and all(np.array_equal(x, wide) for x in out[3:])
    assert np.abs(narrow - wide).max() <= 2e-3


@pytest.mark.parametrize("name,prefix", [("many_kv", 700), ("tiny", 500)])
def test_bits_do_not_depend_on_the_hosts_bound(name, prefix):
    """A window whose length the host only knows a bound of (dropped chunks, uncorrected) takes the same bits as one whose
    length it knows: the key chunks come from the length."""
    shape = S.SHAPES[name]
    toks = S.prefix_tokens(shape, SEED, 0, prefix + 100)
    with _rig(shape, SEED, 2, prefix + 400) as rig:
        for w in (0, 1):
            rig.prefill(w, toks[:prefix])
        for _ in range(4):
            rig.prefill(0, np.full(64, -1))          # not cached: the bound grows, the length stays
        z = [rig.prefill(w, toks[prefix:], want_logits=True) for w in (0, 1)]
        with pytest.raises(dsi.DsiError):
            rig.length(0)                            # the dropped chunks' report
        assert rig.length(0) == rig.length(1) == prefix + 100
        kv = [[rig.export_kv(w, l, prefix + 100) for l in range(shape.n_layers)] for w in (0, 1)]
    assert np.array_equal(*z)
    assert all(np.array_equal(a, b) for x, y in zip(*kv) for a, b in zip(x, y))


@pytest.mark.parametrize("name,n", [("gqa_hd64", 100), ("many_kv", 130)])
def test_captured_prompt_appends_on_every_replay(name, n):
    """A captured prompt that is replayed without a rollback attends to everything before it, past the length it was captured at."""
    import torch
    shape = S.SHAPES[name]
    toks = S.prefix_tokens(shape, SEED, 0, n)
    with torch.cuda.stream(torch.cuda.Stream()), _rig(shape, SEED, 2, 6 * n) as rig:
        rig.prefill(1, toks)                         # reserves what a capture needs
        dsi.dsi_kv_rollback(rig.kv, 1, 0)
        t = rig.dev_i32(toks)
        z = torch.zeros(shape.vocab, device="cuda")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
            dsi.dsi_prefill(rig.model, rig.kv, 0, t, n, z)
        for i in range(5):
            g.replay()
            torch.cuda.synchronize()
            assert rig.length(0) == (i + 1) * n
            want = rig.prefill(1, toks, want_logits=True)
            assert np.abs(z.cpu().numpy() - want).max() <= 2e-3


@pytest.mark.parametrize("name", ["gqa_hd64", "tiny"])
def test_short_calls_captured_after_a_long_prompt(name):
    """A model whose first call is a long prompt: a short prompt and a draft can be captured next, and replay as they run eagerly."""
    import torch
    shape = S.SHAPES[name]
    toks = S.prefix_tokens(shape, SEED, 0, 340)
    with torch.cuda.stream(torch.cuda.Stream()), _rig(shape, SEED, 1, 2000) as rig:
        t = rig.dev_i32(toks)
        u = torch.full((4,), 0.4, device="cuda")
        rig.prefill(0, toks[:300])
        z = torch.zeros(shape.vocab, device="cuda")
        tok, q = torch.zeros(5, dtype=torch.int32, device="cuda"), torch.zeros((4, shape.vocab), device="cuda")

        def calls():
            dsi.dsi_kv_rollback(rig.kv, 0, 240)
            dsi.dsi_prefill(rig.model, rig.kv, 0, t[240:], 40, z)
            dsi.dsi_draft(rig.model, rig.kv, 0, t[280:], 2, 4, u, tok, q)

        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
            calls()
        out = []
        for replay in (True, True, False, True):
            for x in (z, tok, q):
                x.zero_()
            g.replay() if replay else calls()
            torch.cuda.synchronize()
            out.append([x.clone() for x in (z, tok, q)])
    assert bool(out[0][0].any()) and all(torch.equal(a, b) for o in out[1:] for a, b in zip(out[0], o))


def test_captured_launches_outlive_later_prompts():
    """Launches captured before the first wide prompt, replayed after it: it frees nothing that they use."""
    import torch
    shape = S.SHAPES["gqa_hd64"]
    toks = S.prefix_tokens(shape, SEED, 0, 900)
    with torch.cuda.stream(torch.cuda.Stream()), _rig(shape, SEED, 2, 1000) as rig:
        t = rig.dev_i32(toks)
        z = torch.zeros(shape.vocab, device="cuda")
        dsi.dsi_prefill(rig.model, rig.kv, 0, t, 40, z)
        dsi.dsi_kv_rollback(rig.kv, 0, 0)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=torch.cuda.current_stream()):
            dsi.dsi_kv_rollback(rig.kv, 0, 0)
            dsi.dsi_prefill(rig.model, rig.kv, 0, t, 40, z)
        want = None
        for n in (0, 150, 900, 0):
            if n:
                rig.prefill(1, toks[:n])
                dsi.dsi_kv_rollback(rig.kv, 1, 0)
            z.zero_()
            g.replay()
            torch.cuda.synchronize()
            want = z.clone() if want is None else want
            assert torch.equal(z, want) and bool(z.any())
