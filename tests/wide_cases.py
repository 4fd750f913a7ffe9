"""Prompts that between them launch every built variant of the prefill GEMM and
of its fold: (d_model, heads, KV heads, head_dim, d_ff, rows), two layers, bf16
weights.  test_host_runtime.py checks that they do, test_gpu_prefill.py what
they compute."""

WIDE_CASES = [
    # K splits of every role, one row tile and two; QKV and gate/up folded
    (2784, 16, 4, 96, 139, 66), (7936, 64, 8, 96, 401, 35), (4352, 8, 8, 128, 4352, 133), (3680, 32, 4, 128, 1104, 344),
    (6656, 128, 16, 64, 337, 67), (5888, 32, 16, 96, 5888, 205), (2400, 2, 2, 32, 8400, 70), (4096, 8, 1, 32, 11064, 67),
    (8192, 4, 2, 128, 8197, 45),
    # unsplit QKV and gate/up of many row tiles
    (2208, 32, 16, 96, 662, 1156), (256, 64, 8, 32, 691, 1618), (352, 8, 8, 96, 950, 1606), (512, 8, 4, 96, 1792, 1371),
    (768, 128, 16, 64, 2073, 1693), (640, 8, 1, 96, 2240, 1819),
    # and of one (nontemporal weights)
    (320, 128, 16, 64, 864, 58), (2816, 128, 32, 128, 11264, 69), (6144, 40, 40, 96, 24576, 61), (6144, 40, 40, 96, 24576, 66),
    (5024, 32, 16, 32, 40192, 52), (5024, 32, 16, 32, 40192, 80),
]
