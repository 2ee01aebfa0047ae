"""Host-side checks that need no GPU: the library loads, exports what the header declares,
and rejects bad arguments before any HIP call."""
import os
import re

import numpy as np
import pytest

from oracle import lazyllm_oracle as O
from paper_2407_14057_amd import binding as B
from paper_2407_14057_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "lazyllm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(lazyllm_\w+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = B.lib()
    names = _declared_symbols()
    assert len(names) >= 22
    assert lib.lazyllm_op_gemm_workspace_bytes() > 0
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(B._SIGNATURES), "binding and header disagree"
    assert lib.lazyllm_abi_version() == 3
    assert lib.lazyllm_strerror(-1) == b"invalid argument"
    assert lib.lazyllm_strerror(-2) == b"workspace or output buffer too small"
    assert lib.lazyllm_strerror(-5).startswith(b"generation handle unusable")


def test_binding_constants_are_the_headers():
    """Every status code, flag and status bit the header defines has the same value in the binding."""
    text = open(os.path.join(ROOT, "include", "lazyllm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    found = {n: int(v.rstrip("u")) for n, v in re.findall(r"#define\s+(LAZYLLM_\w+)\s+(-?\d+u?)\b", text)}
    found.update({n: int(v) for n, v in re.findall(r"\b(LAZYLLM_E?\w+)\s*=\s*(-?\d+)", text)})
    for name in ("LAZYLLM_OK", "LAZYLLM_EINVAL", "LAZYLLM_ENOSPC", "LAZYLLM_EHIP", "LAZYLLM_ENOMEM", "LAZYLLM_EFAILED",
                 "LAZYLLM_SCORE_ONLY_USED", "LAZYLLM_KEEP_HIDDEN", "LAZYLLM_FUSE_COMPACTION", "LAZYLLM_ST_BAD_TOKEN", "LAZYLLM_ST_BAD_CU",
                 "LAZYLLM_ST_NO_STATE", "LAZYLLM_ST_EXCHANGE"):
        assert name in found, name
        assert getattr(B, name) == found[name], name
    assert found["LAZYLLM_MAX_LAYERS"] == B.MAX_LAYERS
    # the status bits are distinct single bits
    bits = [found[n] for n in found if n.startswith("LAZYLLM_ST_")]
    assert len(bits) == 4 and all(b & (b - 1) == 0 for b in bits) and len(set(bits)) == 4


def test_keep_counts_match_checker():
    cases = [(512, 4, [(2, 700), (3, 500)]), (3376, 32, [(8, 700), (16, 500), (24, 300)]),
             (8192, 32, [(8, 600), (16, 400), (24, 200)]), (3376, 32, [(4, 500), (12, 500), (20, 500)]),
             (10, 3, [(1, 600)]), (1, 5, [(1, 1), (4, 1)]), (7, 4, [(1, 1000), (2, 1)])]
    rng = np.random.default_rng(0)
    for _ in range(50):
        L = int(rng.integers(2, 40))
        layers = sorted(rng.choice(np.arange(1, L), size=min(L - 1, int(rng.integers(1, 5))), replace=False))
        cases.append((int(rng.integers(1, 100000)), L, [(int(l), int(rng.integers(1, 1001))) for l in layers]))
    for n, L, sched in cases:
        assert B.lazyllm_keep_counts(n, L, sched) == O.keep_counts(n, L, sched)


def test_bad_schedules_are_rejected():
    bad = [[(0, 500)],            # layer 0 has no prior scores
           [(4, 500)],            # layer out of range for L = 4
           [(2, 500), (1, 500)],  # unsorted
           [(2, 500), (2, 400)],  # duplicate
           [(1, 0)], [(1, 1001)], [(1, -5)]]
    for sched in bad:
        with pytest.raises(B.LazyLLMError) as e:
            B.lazyllm_keep_counts(100, 4, sched)
        assert e.value.status == B.LAZYLLM_EINVAL
        assert B.lazyllm_output_bytes(B.make_config(synth.TINY.as_dict()), [100], sched) == 0
    with pytest.raises(B.LazyLLMError):
        B.lazyllm_keep_counts(0, 4, [])


def test_sizes_are_positive_and_monotone():
    cfg = B.make_config(synth.TINY.as_dict())
    w1 = B.lazyllm_workspace_bytes(cfg, 512, 1, 512)
    w2 = B.lazyllm_workspace_bytes(cfg, 1024, 2, 512)
    assert 0 < w1 < w2
    o_dense = B.lazyllm_output_bytes(cfg, [512], [])
    o_pruned = B.lazyllm_output_bytes(cfg, [512], [(2, 700), (3, 500)])
    assert o_dense > 0 and o_pruned > 0
    # K/V of layer l hold exactly the tokens that ran it
    kv = lambda counts: sum(2 * n * cfg.d_model * 2 for n in counts)
    assert o_dense >= kv([512] * 4) and o_pruned >= kv([512, 512, 359, 180])
    assert o_pruned < o_dense + 512 * cfg.d_model * 2 + 65536
    # unsupported shapes
    bad = dict(synth.TINY.as_dict())
    bad["head_dim"] = 96
    assert B.lazyllm_workspace_bytes(B.make_config(bad), 512, 1, 512) == 0
    bad = dict(synth.TINY.as_dict())
    bad["n_heads"] = 3
    assert B.lazyllm_workspace_bytes(B.make_config(bad), 512, 1, 512) == 0
    assert B.lazyllm_workspace_bytes(cfg, 0, 1, 1) == 0
    assert B.lazyllm_workspace_bytes(cfg, 10, 1, 11) == 0
    assert B.lazyllm_output_bytes(cfg, [0], []) == 0
    # shared K,V heads: the count must divide the heads and keep the K,V width a multiple of 128
    gqa = dict(synth.TINY.as_dict())
    gqa["n_kv_heads"] = 2
    cfg2 = B.make_config(gqa)
    assert B.lazyllm_workspace_bytes(cfg2, 512, 1, 512) > 0
    assert 0 < B.lazyllm_output_bytes(cfg2, [512], []) < o_dense          # K,V are half as wide
    for bad_kv in (3, 1, 5, -1):                   # 3 does not divide 4; 1 x 64 is not a multiple of 128
        gqa["n_kv_heads"] = bad_kv
        assert B.lazyllm_workspace_bytes(B.make_config(gqa), 512, 1, 512) == 0, bad_kv
    # 8-bit projections: a larger workspace (codes and scales of the activations); shapes whose
    # widths are not multiples of 256 and unknown arithmetic codes are refused
    f8 = dict(synth.TINY.as_dict())
    f8["gemm_dtype"] = 1
    assert B.lazyllm_workspace_bytes(B.make_config(f8), 512, 1, 512) > w1
    assert B.lazyllm_workspace_bytes(B.make_config(synth.TINY_FP8.as_dict()), 512, 1, 512) > w1
    f8["d_model"], f8["n_heads"] = 384, 6
    assert B.lazyllm_workspace_bytes(B.make_config(f8), 512, 1, 512) == 0
    f8 = dict(synth.TINY.as_dict())
    f8["gemm_dtype"] = 2
    assert B.lazyllm_workspace_bytes(B.make_config(f8), 512, 1, 512) == 0


def test_null_arguments_return_einval_without_touching_the_gpu():
    lib = B.lib()
    res = B.lazyllm_result()
    import ctypes as C
    arr, ns = B.make_schedule([(1, 500)])
    assert lib.lazyllm_prefill(None, None, None, 16, arr, ns, 0, None, 0, None, 0, None, C.byref(res)) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_gemm(None, None, None, None, 1, 128, 64, 64, 64, 128, 0, None, 0, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_gemm(1, 1, 1, None, 4, 100, 64, 64, 64, 100, 0, None, 0, None) == B.LAZYLLM_EINVAL   # N % 128
    assert lib.lazyllm_op_gemm(1, 1, 1, None, 4, 128, 60, 64, 64, 128, 0, None, 0, None) == B.LAZYLLM_EINVAL   # K % 64
    assert lib.lazyllm_op_gemm(1, 1, 1, None, 4, 128, 64, 64, 64, 128, 1, None, 0, None) == B.LAZYLLM_EINVAL   # residual w/o R
    assert lib.lazyllm_op_select(1, 10, 0, 1, 1, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_select(1, 10, 11, 1, 1, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_attention(1, 1, 1, 100, 1, 10, 4, 64, None) == B.LAZYLLM_EINVAL             # vt_ld % 64
    assert lib.lazyllm_op_attention(1, 1, 1, 128, 1, 10, 4, 96, None) == B.LAZYLLM_EINVAL             # head_dim
    assert lib.lazyllm_op_score(1, 1, 1, 1, 0, 4, 64, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_score_scratch_bytes(0, 4) == 0
    assert lib.lazyllm_model_create(None, None, None, None) == B.LAZYLLM_EINVAL
    # the 8-bit variant's steps and the weight re-ordering steps
    assert lib.lazyllm_op_quantize_fp8(None, 4, 64, 64, None, 64, None, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_quantize_fp8(16, 4, 60, 64, 16, 64, 16, None) == B.LAZYLLM_EINVAL            # K % 8
    assert lib.lazyllm_op_quantize_fp8(16, 4, 16392, 16392, 16, 16392, 16, None) == B.LAZYLLM_EINVAL   # K > 16384
    assert lib.lazyllm_op_gemm_fp8(None, None, None, None, None, None, 4, 256, 128, 128, 128, 256, 0, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_gemm_fp8(16, 16, 16, 16, 16, None, 4, 128, 128, 128, 128, 128, 0, None) == B.LAZYLLM_EINVAL   # N % 256
    assert lib.lazyllm_op_gemm_fp8(16, 16, 16, 16, 16, None, 4, 256, 64, 64, 64, 256, 0, None) == B.LAZYLLM_EINVAL      # K % 128
    assert lib.lazyllm_op_gemm_fp8(16, 16, 16, 16, 16, None, 4, 256, 128, 128, 128, 256, 1, None) == B.LAZYLLM_EINVAL   # residual w/o R
    assert lib.lazyllm_op_gemm_fp8(24, 16, 16, 16, 16, None, 4, 256, 128, 128, 128, 256, 0, None) == B.LAZYLLM_EINVAL   # alignment
    assert lib.lazyllm_op_pack_weight_ksteps(None, 128, 64, 64, None, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_pack_weight_ksteps(16, 128, 100, 104, 16, None) == B.LAZYLLM_EINVAL         # K % 64
    assert lib.lazyllm_op_pack_weight_stream(16, 100, 64, 64, 16, None) == B.LAZYLLM_EINVAL           # N % 128
    assert lib.lazyllm_op_pack_weight_stream(16, 128, 64, 32, 16, None) == B.LAZYLLM_EINVAL           # stride below K


def test_static_scratch_scoring_validates_before_any_hip_call():
    """The allocation-free Eq. 1 entry point rejects bad arguments and sizes beyond its static
    scratch on the host (no GPU here: reaching a HIP call would fail differently)."""
    lib = B.lib()
    one = 4096
    assert lib.lazyllm_op_score_static(None, one, one, 10, 4, 64, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_score_static(one, one, one, 0, 4, 64, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_score_static(one, one, one, 10, 4, 96, None) == B.LAZYLLM_EINVAL
    assert lib.lazyllm_op_score_static(one, one, one, 40000, 64, 128, None) == B.LAZYLLM_ENOSPC
    # the limit is the scratch size the buffer form would ask for
    assert B.lazyllm_op_score_scratch_bytes(39000, 32) <= 6 * 1024 * 1024 < B.lazyllm_op_score_scratch_bytes(40000, 32)
    assert lib.lazyllm_op_score_static(one, one, one, 40000, 32, 128, None) == B.LAZYLLM_ENOSPC


def test_bench_refuses_more_than_one_gpu():
    """One GPU is the whole target: `bench.py --gpus N` with N above 1 says so and exits non-zero,
    before anything touches a device."""
    import subprocess, sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


# the tiles gemm_stream.hip builds; three- and four-wave tiles of two or four row blocks: one row chunk only
_BUILT = {(2, 2, 4), (4, 2, 4), (8, 2, 4), (2, 3, 2), (4, 3, 2), (2, 4, 2), (4, 4, 2), (6, 3, 2), (8, 3, 2), (6, 4, 2), (8, 4, 2),
          (6, 6, 1), (8, 6, 1), (8, 8, 1), (6, 12, 1), (8, 12, 1), (10, 12, 1)}
_MODELS = {"7b": (4096, 4096, 11008), "grouped query 8b": (4096, 1024, 14336), "narrow": (1280, 1280, 3456), "2048": (2048, 512, 8192),
           "3072": (3072, 1024, 8192), "5120": (5120, 5120, 13824), "8192": (8192, 1024, 28672), "tiny": (256, 256, 768), "1024": (1024, 1024, 2816)}


def _projections(d, kv, ffn):
    return [(d + 2 * kv, d), (d, d), (2 * ffn, d), (d, ffn)]


def test_streaming_plan_returns_tiles_that_are_built():
    for d, kv, ffn in _MODELS.values():
        for N, K in _projections(d, kv, ffn):
            for M in range(1, 700):
                p = B.lazyllm_op_gemm_stream_plan(M, N, K)
                if p is None:
                    assert M > 32, (M, N, K)                 # few rows always stream
                    continue
                tm, cw, kw, ks = p
                assert (tm, cw, kw) in _BUILT, (M, N, K, p)
                assert ks >= 1 and ks * kw <= max(K // 64, kw), (M, N, K, p)
                assert cw % 3 == 0 or N % (cw * 32) == 0, (M, N, K, p)
                if cw in (3, 4) and tm in (2, 4):
                    assert M <= tm * 16, (M, N, K, p)
    assert B.lazyllm_op_gemm_stream_plan(0, 4096, 4096) is None
    assert B.lazyllm_op_gemm_stream_plan(1, 4000, 4096) is None and B.lazyllm_op_gemm_stream_plan(1, 4096, 100) is None
    assert B.lib().lazyllm_op_gemm_stream_plan(1, 128, 64, None) == B.LAZYLLM_EINVAL
    # a forced streaming launch beyond the rule is refused before the device is touched
    assert B.lib().lazyllm_op_gemm(16, 16, 16, None, 641, 128, 1088, 1088, 1088, 128, 8 << 8, 256, 1 << 30, None) == B.LAZYLLM_EINVAL


def test_streaming_plan_of_a_short_k_ends_after_one_round_of_the_compute_units():
    """K up to 1024: whatever the widths, no more workgroups than the 32 compute units of an XCD hold at
    once, beyond that the tile kernels (twice to three times as fast from a few rounds on).  The one
    exception is a K of one step, up to the row count for which packed prompts keep their own bits."""
    for d, kv, ffn in [(256, 256, 768), (512, 512, 960), (768, 768, 1024), (1024, 1024, 1024), (1024, 256, 4096)]:
        for N, K in _projections(d, kv, ffn):
            if K > 1024:
                continue
            taken = 0
            for M in list(range(1, 600)) + list(range(600, 17000, 37)):
                p = B.lazyllm_op_gemm_stream_plan(M, N, K)
                if p is None:
                    continue
                taken = M
                per_xcd = -(-(N // 64) // 8) * -(-M // (p[0] * 16))
                assert M <= 32 or per_xcd <= 32 or (K <= 256 and M <= 3200), (M, N, K, p, per_xcd)
            assert 128 <= taken <= 3584, (N, K, taken)
    for M, N, K in [(2048, 8192, 1024), (8192, 1024, 1024), (1536, 1536, 512), (4096, 256, 256), (16384, 256, 768), (3201, 768, 256)]:
        assert B.lazyllm_op_gemm_stream_plan(M, N, K) is None, (M, N, K)
    # the packed batch of a thousand short prompts and each of its prompts: the same kernel, the same order of sums
    for N, K in _projections(256, 256, 768):
        assert B.lazyllm_op_gemm_stream_plan(3094, N, K)[1:] == B.lazyllm_op_gemm_stream_plan(5, N, K)[1:]


def test_streaming_plan_has_no_holes_in_the_rows_of_the_shipped_models():
    """Once the tile kernels take a projection of the 4096-wide models, they take it at every larger row count."""
    for d, kv, ffn in (_MODELS["7b"], _MODELS["grouped query 8b"]):
        for N, K in _projections(d, kv, ffn):
            taken = [M for M in range(1, 900) if B.lazyllm_op_gemm_stream_plan(M, N, K) is not None]
            assert taken == list(range(1, len(taken) + 1)), (N, K, [a for a, b in zip(taken, taken[1:]) if b != a + 1])
            assert len(taken) == (480 if N == 28672 else 640)
    for M in (289, 355, 384):
        assert B.lazyllm_op_gemm_stream_plan(M, 28672, 4096) == (8, 12, 1, 1)


def test_streaming_plan_leaves_out_the_tiles_that_lose_to_the_tile_kernels():
    plan = B.lazyllm_op_gemm_stream_plan
    for N in (24704, 26752, 30848):                          # half the chip idle on twelve waves
        for M in (129, 160, 200, 256):
            assert plan(M, N, 4096) is None, (M, N)
    assert plan(257, 15488, 2048) is None and plan(257, 24704, 4096) == (6, 12, 1, 1) and plan(257, 22016, 4096) == (6, 12, 1, 1)
    for N, K in ((4352, 11008), (5120, 8192), (5120, 13824)):
        assert all(plan(M, N, K) is None for M in range(289, 385)) and plan(288, N, K) is not None and plan(385, N, K) is not None
    for N in (256, 512, 768):
        for K in (1088, 1408):
            assert all(plan(M, N, K)[2] > 1 for M in range(385, 641))
    assert plan(65, 8192, 28672) == (6, 4, 2, 4)


def test_decode_key_splits_leave_no_wide_step_on_one_range():
    """Workgroups of a step's attention (heads x blocks of 128 rows x key ranges): one full round of the 256
    compute units, else about two per unit; never a single range of a long sequence while the workspace
    holds another, which took 1.3 to 1.7 times as long."""
    splits = B.lib().lazyllm_op_decode_key_splits
    assert [splits(m, 4096, 32, 128) for m in (2, 128, 129, 256, 384, 512, 640, 768, 1024, 1025)] == [8, 8, 4, 4, 5, 2, 3, 2, 2, 1]
    assert [splits(m, 2048, 32, 128) for m in (128, 256, 384, 512, 640, 768, 1024)] == [8, 4, 5, 2, 3, 2, 1]
    assert [splits(m, 1024, 32, 128) for m in (128, 256, 384, 512)] == [8, 4, 2, 2]
    assert [splits(m, 4096, 40, 128) for m in (128, 256, 384, 512, 640)] == [6, 3, 2, 3, 2]
    for heads, hd in ((4, 64), (8, 64), (32, 128), (40, 128), (64, 128)):
        for keys in (64, 700, 1500, 2500, 4096, 8192):
            for m in range(2, 2049, 7):
                n, base, tiles = splits(m, keys, heads, hd), heads * -(-m // 128), (keys + 63) // 64
                assert 1 <= n <= 16 and (n == 1 or n <= tiles // 2), (heads, keys, m, n)
                assert n == 1 or n * m <= 16 * 128, (heads, keys, m, n)          # what the workspace holds
                if keys > 2048 and base <= 256 and 2 * m <= 16 * 128:
                    assert n > 1, (heads, keys, m)
    assert splits(1, 64, 4, 64) == B.LAZYLLM_EINVAL and splits(2, 0, 4, 64) == B.LAZYLLM_EINVAL and splits(2, 64, 4, 96) == B.LAZYLLM_EINVAL


def test_attention_form_counts_the_whole_batch():
    """Shared keys while all sequences together make at most one workgroup per compute unit (two with 64-wide
    heads): beyond it that form took 1.2 to 2 times as long, whatever the number of heads.  With one key step
    it is the smaller workgroup of the two."""
    block = B.lib().lazyllm_op_attention_block
    for heads in (1, 2, 4, 8, 16, 32):
        for hd, limit in ((64, 512), (128, 256)):
            for rows in (65, 97, 180, 256, 512, 1024, 2048):
                for batch in (1, 2, 3, 8, 64, 1000):
                    shared = -(-rows // 32) * heads * batch
                    assert (block(rows, batch, heads, hd) == 32) == (shared <= limit), (rows, batch, heads, hd)
    assert [block(n, 1000, 4, 64) for n in (5, 32, 33, 64, 65)] == [32, 32, 32, 32, 256]
    assert [block(n, 64, 8, 128) for n in (5, 32, 33)] == [32, 32, 256] and block(33, 256, 8, 128) == 32 and block(5, 8, 8, 128) == 128
    assert block(512, 1, 4, 64) == 32 and block(3376, 1, 32, 128) == 256 and block(844, 1, 32, 128) == 128
    for bad in ((0, 1, 4, 64), (8, 0, 4, 64), (8, 1, 0, 64), (8, 1, 4, 96)):
        assert block(*bad) == B.LAZYLLM_EINVAL


def test_forced_8bit_configurations_that_do_not_fit_are_refused_before_the_device_is_touched():
    call = B.lib().lazyllm_op_gemm_fp8_ws
    big = 1 << 30
    args = (16, 16, 16, 16, 16, None, 64, 256, 128, 128, 128, 256)
    for cfg in (1, 3, 4, 6, 8, 11, 14, 17, 255):
        assert call(*args, cfg << 8, 256, big, None) == B.LAZYLLM_EINVAL, cfg
    for cfg in (9, 10, 16):                                  # stream-K without a (large enough) workspace
        assert call(*args, cfg << 8, None, 0, None) == B.LAZYLLM_EINVAL
        assert call(*args, cfg << 8, 256, 4096, None) == B.LAZYLLM_EINVAL
    assert call(*args, 0, 128, big, None) == B.LAZYLLM_EINVAL        # workspace not on a 256-byte boundary
    # the entry point without a workspace takes no configuration
    for cfg in (2, 5, 9):
        assert B.lib().lazyllm_op_gemm_fp8(*args, cfg << 8, None) == B.LAZYLLM_EINVAL
    for plan, bad in ((B.lib().lazyllm_op_gemm_fp8_plan, (8, 128, 128, 0, 0)), (B.lib().lazyllm_op_gemm_fp8_plan, (8, 256, 64, 0, 0)),
                      (B.lib().lazyllm_op_gemm_fp8_plan, (0, 256, 128, 0, 0)), (B.lib().lazyllm_op_gemm_plan, (8, 64, 64, 0, 0, 0)),
                      (B.lib().lazyllm_op_gemm_plan, (8, 128, 64, 3, 96, 0)), (B.lib().lazyllm_op_gemm_plan, (8, 128, 64, 0, 0, 4))):
        assert plan(*bad) == B.LAZYLLM_EINVAL


def test_tile_choice_at_shapes_where_an_estimate_was_off():
    """Shapes at which the estimated times once picked a form 8 to 23 % behind the best: one of the forms measured
    within 3 % of the best must be chosen (16-bit with a workspace, 8-bit likewise)."""
    for (M, N, K, epi, hd), good in {
            (1182, 6144, 4096, 3, 128): (15,), (6384, 2304, 768, 3, 64): (5,), (12288, 2304, 768, 3, 64): (5,),
            (703, 8192, 1536, 2, 64): (2, 15), (645, 2560, 6912, 1, 128): (6,), (704, 22016, 4096, 2, 128): (10,),
            (768, 22016, 4096, 2, 128): (10,), (991, 22016, 4096, 2, 128): (9,)}.items():
        assert B.lib().lazyllm_op_gemm_plan(M, N, K, epi, hd, 1) in good, (M, N, K, epi)
    for (M, N, K, epi), good in {
            (86, 16384, 3072, 2): (2,), (186, 32768, 6144, 2): (2,), (26, 27648, 5120, 2): (2,), (45, 12288, 4096, 3): (2,),
            (281, 2048, 5504, 1): (2, 15)}.items():
        assert B.lib().lazyllm_op_gemm_fp8_plan(M, N, K, epi, 1) in good, (M, N, K, epi)


def test_small_models_do_not_split_k_over_workgroups():
    """A model 256 wide: no tile of any row count adds its sums in pieces, so that a packed prompt's projections
    have the bits of the prompt alone."""
    for N, K, epi in ((768, 256, 3), (256, 256, 1), (1536, 256, 2), (256, 768, 1)):
        for M in list(range(1, 400)) + list(range(400, 16385, 61)):
            assert B.lib().lazyllm_op_gemm_plan(M, N, K, epi, 64, 3) not in (6, 9, 10, 16), (M, N, K)
            assert B.lib().lazyllm_op_gemm_fp8_plan(M, N, K, epi, 1) not in (9, 10, 16), (M, N, K)


_CLEAN_ASM = """kernel:
\tds_read_b128 v[0:3], v40
\ts_waitcnt lgkmcnt(0)
\t;;#ASMSTART
\tv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[8:11], a[0:3]
\t;;#ASMEND
\t;;#ASMSTART
\tv_accvgpr_read_b32 v5, a7
\t;;#ASMEND
\tv_add_f32_e32 v6, v5, v4
\ts_endpgm
    .private_segment_fixed_size: 0
    .vgpr_spill_count: 0
"""


@pytest.mark.parametrize("ahead,what", [
    ("v_accvgpr_write_b32 a7, v4", "accumulation register"), ("v_add_f32_e32 v30, a[3:4], v2", "accumulation register"), ("v_add_f32_e32 v30, a3, v2", "accumulation register"),
    ("ds_read_b128 a[12:15], v40", "accumulation register"), ("global_store_dwordx4 v[20:21], a[0:3], off", "accumulation register"),
    ("v_mov_b32_e32 v9, v4", "0 wait states"), ("v_mov_b32_e32 v9, v4\n\ts_nop 0", "1 wait states"), ("v_mov_b32_e32 v9, v4\n\ts_nop 1", None),
    ("v_pk_mul_f32 v[2:3], v[2:3], v[4:5]\n\tv_mov_b32_e32 v30, v4", "1 wait states"), ("v_mov_b32_e32 v12, v0", None),
    ("v_cmp_gt_f32_e32 vcc, v0, v8", None), ("ds_read_b128 v[0:3], v40", None), ("s_mov_b32 s0, s1", None),
    ("    .vgpr_spill_count: 2", "vgpr_spill_count"), ("    .private_segment_fixed_size: 16", "private_segment")])
def test_build_looks_for_what_could_corrupt_named_accumulators(ahead, what):
    """The check that the build runs on the assembly of the kernels whose accumulators are named registers."""
    from paper_2407_14057_amd.build import accumulator_faults
    assert accumulator_faults(_CLEAN_ASM) == []
    at = _CLEAN_ASM.index("\t;;#ASMSTART")
    faults = accumulator_faults(_CLEAN_ASM[:at] + ("" if ahead.startswith(" ") else "\t") + ahead + "\n" + _CLEAN_ASM[at:])
    if what is None:
        assert faults == [], faults
    else:
        assert len(faults) == 1 and what in faults[0], faults
