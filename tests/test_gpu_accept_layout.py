"""The accept/reject kernels on every load path: vocabularies at the edges of a
chunk (4096 entries) and of a thread's four entries, row buffers that are
16-byte aligned or not, few and many (row, chunk) pairs, masked logits."""
import numpy as np
import pytest
import torch

from paper_2405_14105_amd import dsi
from test_gpu_accept import _inputs, compare

pytestmark = pytest.mark.gpu


def _at(a, off):
    """The array on the GPU, `off` elements into its buffer."""
    buf = torch.zeros(a.size + 4, dtype=torch.float32, device="cuda")
    buf[off:off + a.size] = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32).reshape(-1))
    return buf, buf.data_ptr() + 4 * off


@pytest.mark.parametrize("V,B,k", [(1, 3, 2), (4095, 2, 3), (4096, 2, 3), (4097, 2, 3), (4100, 16, 3), (40000, 16, 3),
                                   (40001, 60, 0), (36868, 4, 12)])
@pytest.mark.parametrize("zoff,qoff", [(0, 0), (1, 0), (0, 2)])
@pytest.mark.parametrize("T", [1.0, 0.7])
def test_layouts(V, B, k, zoff, qoff, T):
    z, tokens, q, u = _inputs(V, k, B, seed=V + 7 * k)
    if V > 8:                                  # a tenth of the entries masked, never a draft
        mask = np.random.default_rng(V).random(z.shape) < 0.1
        for b in range(B):
            for i in range(k):
                mask[b * (k + 1) + i, tokens[b, i + 1]] = False
        z[mask] = -np.inf
    zb, zp = _at(z, zoff)
    qb, qp = _at(q if k else np.zeros(1), qoff)
    t = torch.from_numpy(np.ascontiguousarray(tokens, dtype=np.int32)).cuda()
    du = torch.from_numpy(np.ascontiguousarray(u, dtype=np.float32)).cuda()
    n = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    tok = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    dsi.dsi_accept(torch.cuda.current_stream().cuda_stream, B, k, V, zp, t, qp if k else None, du, n, tok, T,
                   dsi.DSI_SAMPLE)
    torch.cuda.synchronize()
    assert compare(z, tokens, q, u, n.cpu().numpy(), tok.cpu().numpy(), T=T) <= max(1, B // 10)
    # each window alone: the same decision
    for b in range(min(B, 4)):
        n1 = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        t1 = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        dsi.dsi_accept(torch.cuda.current_stream().cuda_stream, 1, k, V, zp + 4 * b * (k + 1) * V, t[b],
                       qp + 4 * b * k * V if k else None, du[b], n1, t1, T, dsi.DSI_SAMPLE)
        torch.cuda.synchronize()
        assert (int(n1), int(t1)) == (int(n[b]), int(tok[b]))


@pytest.mark.parametrize("V,keep", [(4100, (0, 4096)), (40000, (4096, 40000)), (40000, (20000, 20050)), (12288, (0, 8192)),
                                    (128256, (100000, 128000))])
@pytest.mark.parametrize("B,k", [(2, 3), (16, 3)])
def test_whole_chunks_masked(V, keep, B, k):
    """Only the entries of [keep) are not -inf: first, middle and last chunks, all but one of them, a tail of four entries."""
    z, tokens, q, u = _inputs(V, k, B, seed=V + keep[0] + k)
    rng = np.random.default_rng(V)
    tokens[:, 1:] = rng.integers(*keep, size=(B, k))
    z[:, :keep[0]] = -np.inf
    z[:, keep[1]:] = -np.inf
    for b in range(B):                         # every draft at the target's own probability: accepted with ratio > u
        for i in range(k):
            p = z[b * (k + 1) + i, tokens[b, i + 1]] - np.log(np.exp(z[b * (k + 1) + i, keep[0]:keep[1]].astype(np.float64)).sum())
            q[b, i, tokens[b, i + 1]] = np.exp(p) * (0.5 if (b + i) % 3 else 4.0)
    n = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    tok = torch.full((B,), -7, dtype=torch.int32, device="cuda")
    dev = [torch.from_numpy(np.ascontiguousarray(x, dtype=d)).cuda() for x, d in
           ((z, np.float32), (tokens, np.int32), (q, np.float32), (u, np.float32))]
    dsi.dsi_accept(torch.cuda.current_stream().cuda_stream, B, k, V, *dev, n, tok, 1.0, dsi.DSI_SAMPLE)
    torch.cuda.synchronize()
    n, tok = n.cpu().numpy(), tok.cpu().numpy()
    assert np.all((tok >= keep[0]) & (tok < keep[1])) and n.max() > 0
    assert compare(z, tokens, q, u, n, tok) <= max(1, B // 10)
