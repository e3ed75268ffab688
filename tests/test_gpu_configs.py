"""GPU parity at the five benchmark configurations, full size, through the C ABI."""
import numpy as np
import pytest

import oracle
import vq_synth as s
from cases import lent

pytestmark = pytest.mark.gpu
TOL = 1e-2


@pytest.fixture(scope="module")
def layers():
    cache = {}

    def get(cfg, name=None):
        key = (cfg, name)
        if key not in cache:
            cache.clear()                      # one big layer resident at a time
            cache[key] = next(s.config_layers(cfg, only=name))
        return cache[key]
    return get


def _dequant_exact(gpu_lib, L):
    import torch
    dl = gpu_lib.DeviceLayer(L)
    W = gpu_lib.dequant(dl)
    torch.cuda.synchronize()
    got = W.cpu().numpy().view(np.uint16)
    del W
    want = oracle.dequant(L).view(np.uint16)
    assert np.array_equal(got, want)
    return dl


def _matmul_ok(y, ref, what):
    y = y.float().cpu().numpy().astype(np.float64)
    rms = np.sqrt((ref ** 2).mean())
    err = np.abs(y - ref).max()
    assert np.isfinite(y).all() and err <= TOL * rms, "%s: err %.3e rms %.3e" % (what, err, rms)


@pytest.mark.parametrize("cfg,name", [(0, "tiny"), (1, "up"), (2, "q"), (2, "o"), (2, "gate"), (2, "down"), (3, "down70b"), (4, "prefill")])
def test_config_dequant_and_gemv(gpu_lib, layers, monkeypatch, cfg, name):
    import torch
    ordinal, L = layers(cfg, name)
    dl = _dequant_exact(gpu_lib, L)
    spec = s.CONFIGS[cfg]
    batches = spec["rows"] if cfg != 4 else [1, 16]
    for batch in batches:
        x = s.make_activations(cfg, L, batch, layer_ordinal=ordinal, outlier_gain=spec.get("outlier_gain", 1.0))
        ref = oracle.gemv(L, x)
        xd = torch.from_numpy(x).cuda()
        for kernel in ("auto", "m", "d"):              # default dispatch, matrix-core kernel, dot-product kernels
            if kernel != "auto":
                monkeypatch.setenv("VQ_SWITCHES", "gemv=" + kernel)
            y = gpu_lib.gemv(dl, xd)
            torch.cuda.synchronize()
            monkeypatch.delenv("VQ_SWITCHES", raising=False)
            _matmul_ok(y, ref, "cfg%d %s batch %d kernel %s" % (cfg, name, batch, kernel))


@pytest.mark.parametrize("tokens", [512, 1024, 2048])
@pytest.mark.parametrize("workspace", [None, "none", "fast"])
def test_config4_prefill_gemm(gpu_lib, layers, tokens, workspace):
    import torch
    _, L = layers(4, "prefill")
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(4, L, tokens)
    Y = gpu_lib.gemm(dl, torch.from_numpy(x).cuda(), workspace=lent(workspace))
    torch.cuda.synchronize()
    if tokens == 512:
        _matmul_ok(Y, oracle.gemm(L, x), "cfg4 T=512 full")
    else:
        # larger token counts: every 16th output row plus the edges, all tokens
        rows = np.unique(np.concatenate([np.arange(0, L.out_features, 16), [L.out_features - 1, 127, 128, 8191 - 128]])).astype(np.int32)
        ref = oracle.gemm(L, x, rows=rows)
        _matmul_ok(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()], ref, "cfg4 T=%d sampled rows" % tokens)


@pytest.mark.parametrize("workspace", [None, "none", "fast"])
def test_config3_small_gemm_with_outliers(gpu_lib, layers, workspace):
    import torch
    _, L = layers(3, "down70b")
    sub = s.make_layer(3, "slice", 256, L.in_features, 6, 4096, 256, 288, 4, 4096)
    dl = gpu_lib.DeviceLayer(sub)
    x = s.make_activations(3, sub, 64, outlier_gain=10.0)
    Y = gpu_lib.gemm(dl, torch.from_numpy(x).cuda(), workspace=lent(workspace))
    torch.cuda.synchronize()
    _matmul_ok(Y, oracle.gemm(sub, x), "cfg3 slice gemm")


@pytest.mark.parametrize("names", [("q", "k", "v"), ("gate", "up")])
def test_config2_projections_in_one_launch(gpu_lib, names):
    """vq_gemv_multi as the benchmark runs it: the 7B decoder layer's q, k, v (and gate, up) on one x, every output row."""
    import torch
    pairs = [next(s.config_layers(2, only=n)) for n in names]
    dls = [gpu_lib.DeviceLayer(L) for _, L in pairs]
    for batch in s.CONFIGS[2]["rows"]:
        x = s.make_activations(2, pairs[0][1], batch, layer_ordinal=pairs[0][0])
        ys = gpu_lib.gemv_multi(dls, torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        for (_, L), y in zip(pairs, ys):
            _matmul_ok(y, oracle.gemv(L, x), "cfg2 %s of %s batch %d" % (L.name, "+".join(names), batch))


@pytest.mark.parametrize("group_vectors", [176, 48])
def test_headline_shape_with_codebook_groups(gpu_lib, group_vectors):
    """The 11008 x 4096 layer split into 4 and 15 codebook groups, as bench.py's detail lines time it."""
    import torch
    L = s.make_layer(1, "up", 11008, 4096, 6, 4096, group_vectors=group_vectors)
    dl = _dequant_exact(gpu_lib, L)
    for batch in (1, 16):
        x = s.make_activations(1, L, batch)
        ref = oracle.gemv(L, x)
        for workspace in ("none", "fast"):
            y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda(), workspace=lent(workspace))
            torch.cuda.synchronize()
            _matmul_ok(y, ref, "grouped headline shape, %d vectors a group, batch %d, workspace %s" % (group_vectors, batch, workspace))


@pytest.mark.parametrize("extra", [dict(), dict(k_res=4096, n_outlier_cols=40, v_out=4, k_out=4096), dict(group_vectors=256, k_res=256)])
def test_headline_shape_in_the_papers_orientation(gpu_lib, extra):
    """The 11008 x 4096 layer with vectors down the output dimension, as bench.py's detail lines time it: the vector-ALU
    kernel (one row), the matrix-core kernel alone and with the column parts of the workspace route."""
    import torch
    L = s.make_layer(1, "up", 11008, 4096, 6, 4096, orientation=1, **extra)
    dl = _dequant_exact(gpu_lib, L)
    for batch in (1, 4, 7, 16):
        x = s.make_activations(1, L, batch)
        ref = oracle.gemv(L, x)
        for workspace in ("none", "fast"):
            y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda(), workspace=lent(workspace))
            torch.cuda.synchronize()
            _matmul_ok(y, ref, "headline shape, orientation 1, batch %d, %s, workspace %s" % (batch, extra, workspace))


def test_config3_with_scattered_outlier_columns(gpu_lib):
    """The 8192 x 28672 layer of the 70B setting with its columns stored in a permuted order, so that the 288 outlier
    columns lie scattered over the layer (Sec. 3.2.3): restored matrix bit-exact, products with and without a workspace."""
    import torch
    c = s.CONFIGS[3]
    L = s.make_layer(3, "down70b", 8192, 28672, c["v"], c["k"], c["k_res"], c["n_outlier_cols"], c["v_out"], c["k_out"], permute=True)
    assert sorted(L.col_perm[:288]) != list(range(288))
    dl = _dequant_exact(gpu_lib, L)
    for batch in (1, 8):
        x = s.make_activations(3, L, batch, outlier_gain=c["outlier_gain"])
        ref = oracle.gemv(L, x)
        for workspace in ("none", "fast"):
            y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda(), workspace=lent(workspace))
            torch.cuda.synchronize()
            _matmul_ok(y, ref, "cfg3 with permuted columns, batch %d, workspace %s" % (batch, workspace))


@pytest.mark.parametrize("cfg,name,tokens", [(1, "up", 512), (2, "q", 300), (2, "down", 130), (3, "down70b", 130)])
def test_prefill_without_workspace_on_the_v6_layers(gpu_lib, layers, cfg, name, tokens):
    """vq_gemm without a workspace on the 7B-shaped v = 6 layers (no residual; 12-bit residual) and on the 70B-shaped one (8-bit
    residual, 288 outlier columns): the kernel that restores W on the fly from tables in LDS, every 16th output row plus the
    edges against the oracle."""
    import torch
    ordinal, L = layers(cfg, name)
    dl = gpu_lib.DeviceLayer(L)
    assert gpu_lib.vq_gemm_workspace_bytes(dl.desc, tokens) == 0
    x = s.make_activations(cfg, L, tokens, layer_ordinal=ordinal)
    Y = gpu_lib.gemm(dl, torch.from_numpy(x).cuda(), workspace=lent("none"))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, L.out_features, 16), [L.out_features - 1, 127, 128, L.out_features - 128]])).astype(np.int32)
    _matmul_ok(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()], oracle.gemm(L, x, rows=rows), "cfg%d %s T=%d on the fly" % (cfg, name, tokens))


@pytest.mark.parametrize("out,inp,k", [(14341, 4104, 65536), (7371, 8200, 65530), (20480, 3072, 40000)])
def test_long_prompts_of_the_v8_setting_restore_the_same_weights(gpu_lib, out, inp, k):
    """In front of a product of many tokens a layer of v = 8 with a table beyond LDS is restored by a kernel of its own: the weights that it
    leaves in the workspace are vq_dequant's, bit for bit (which the oracle checks elsewhere, and here on a few rows)."""
    import torch
    L = s.make_layer(4, "pieces", out, inp, 8, k)
    dl = gpu_lib.DeviceLayer(L)
    size = gpu_lib.vq_gemm_fast_workspace_bytes(dl.desc, 1024)
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
    x = torch.randn((1024, inp), device="cuda").half()
    Y = gpu_lib.gemm(dl, x, workspace=ws)
    W = gpu_lib.dequant(dl)
    torch.cuda.synchronize()
    assert torch.equal(ws[: out * inp * 2].view(torch.int16), W.view(torch.int16).reshape(-1))
    rows = np.array([0, 1, out // 2, out - 1], dtype=np.int32)
    _matmul_ok(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()][:64], oracle.gemm(L, x[:64].cpu().numpy(), rows=rows), "v8 %d x %d, 1024 tokens" % (out, inp))


@pytest.mark.parametrize("out,inp,tokens,permute,setting", [
    (8191, 16000, 1024, False, dict(v=8, k=65536)),              # W of 262 MB: past the caches, from the pieces of the table
    (7903, 4104, 1024, False, dict(v=8, k=40000)),               # a single turn of all workgroups, just full enough
    (7371, 8200, 1024, True, dict(v=8, k=65536)),                # permuted columns: the gathered activations lie in front of W
    (9003, 584, 40, False, dict(v=8, k=65536)),                  # a short product of short rows: past the caches
    (9001, 592, 130, False, dict(v=12, k=4096, k_res=4096)),
    (9003, 584, 200, True, dict(v=8, k=65536, k_res=256)),       # more tokens: through them
])
def test_restoring_in_front_of_a_product_leaves_the_same_weights(gpu_lib, out, inp, tokens, permute, setting):
    """What vq_gemm restores into its workspace is what vq_dequant restores from the layer in stored order, bit for bit, whichever way the
    stores go; and the product is that of a few rows."""
    import torch
    L = s.make_layer(5, "front", out, inp, permute=permute, **setting)
    dl = gpu_lib.DeviceLayer(L)
    size = gpu_lib.vq_gemm_fast_workspace_bytes(dl.desc, tokens)
    head = (tokens * inp * 2 + 255) // 256 * 256 if permute else 0
    assert size >= head + out * inp * 2
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
    x = torch.randn((tokens, inp), device="cuda").half()
    Y = gpu_lib.gemm(dl, x, workspace=ws)
    rows = np.array([0, 1, out // 2, out - 1], dtype=np.int32)
    ref = oracle.gemm(L, x[:16].cpu().numpy(), rows=rows)
    L.col_perm = None
    W = gpu_lib.dequant(gpu_lib.DeviceLayer(L))
    torch.cuda.synchronize()
    assert torch.equal(ws[head : head + out * inp * 2].view(torch.int16), W.view(torch.int16).reshape(-1))
    _matmul_ok(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()][:16], ref, "%d x %d, %d tokens" % (out, inp, tokens))


# Rows for which a workgroup of the matrix-core kernel has 4, 5, 6 and 7 blocks of sixteen (256 compute units): one chunk over the tables
# where its partial sums do not fit beside them, one beside them, and two chunks of four and three blocks.
@pytest.mark.parametrize("out,k_res,outliers", [(12300, 4096, 0), (16400, 0, 0), (20480, 256, 8), (24560, 4096, 8), (24561, 256, 0), (24592, 4096, 0)])
def test_many_blocks_a_workgroup(gpu_lib, out, k_res, outliers):
    import torch
    L = s.make_layer(1, "up", out, 391, 6, 4096, k_res, **(dict(n_outlier_cols=outliers, v_out=4, k_out=4096) if outliers else {}))
    dl = gpu_lib.DeviceLayer(L)
    second = s.make_layer(2, "up", 70, 391, 6, 4096, k_res)
    for batch in (3, 16):
        x = s.make_activations(1, L, batch)
        ref = oracle.gemv(L, x)
        xd = torch.zeros((batch, 392), dtype=torch.float16, device="cuda")
        xd[:, :391] = torch.from_numpy(x)
        y = gpu_lib.gemv(dl, xd[:, :391], workspace=lent("none"))
        ym, ys = gpu_lib.gemv_multi([dl, gpu_lib.DeviceLayer(second)], xd[:, :391])
        torch.cuda.synchronize()
        _matmul_ok(y, ref, "%d rows, k_res %d, batch %d" % (out, k_res, batch))
        _matmul_ok(ym, ref, "%d rows, k_res %d, batch %d, one of two" % (out, k_res, batch))
        _matmul_ok(ys, oracle.gemv(second, x), "70 rows beside %d, k_res %d, batch %d" % (out, k_res, batch))


@pytest.mark.parametrize("orientation", [0, 1])
def test_the_2_26_bit_setting_at_full_size(gpu_lib, orientation):
    """The 11008 x 4096 layer in the 2.26-bit setting of Table "Quantization parameters" (v = 12, two 4096-entry tables, four
    codebook groups, 40 outlier columns of v = 4 with 8192 entries), both orientations: vq_dequant bit for bit, vq_gemv with one
    and with five rows, without and with a workspace, vq_gemm at 300 tokens through the restore-then-multiply route on every
    16th output row."""
    import torch
    P = -(-(4096 - 40) // 12) if orientation == 0 else 4096 - 40
    L = s.make_layer(1, "up", 11008, 4096, 12, 4096, 4096, n_outlier_cols=40, v_out=4, k_out=8192, group_vectors=-(-P // 4),
                     orientation=orientation)
    dl = _dequant_exact(gpu_lib, L)
    for batch in (1, 5):
        x = s.make_activations(1, L, batch)
        ref = oracle.gemv(L, x)
        for workspace in ("none", "fast"):
            y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda(), workspace=lent(workspace))
            torch.cuda.synchronize()
            _matmul_ok(y, ref, "2.26-bit setting, orientation %d, batch %d, workspace %s" % (orientation, batch, workspace))
    x = s.make_activations(1, L, 300)
    Y = gpu_lib.gemm(dl, torch.from_numpy(x).cuda(), workspace="fast")
    torch.cuda.synchronize()
    rows = np.arange(0, L.out_features, 16).astype(np.int32)
    _matmul_ok(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()], oracle.gemm(L, x, rows=rows), "2.26-bit setting, 300 tokens")


@pytest.mark.parametrize("out,inp", [(11008, 4096), (4096, 11008)])
def test_one_row_of_the_2_26_bit_setting_takes_no_longer_than_two(gpu_lib, out, inp):
    """Without a workspace both go through the kernel that keeps one table in LDS at a time, and two rows do all that one does
    and the products of the second besides (41 and 49 us for 11008 x 4096)."""
    import torch
    n_out = int(inp * 0.01 / 4 + 0.5) * 4
    P = -(-(inp - n_out) // 12)
    L = s.make_layer(1, "up", out, inp, 12, 4096, 4096, n_outlier_cols=n_out, v_out=4, k_out=8192, group_vectors=-(-P // 32) * 8)
    dl = gpu_lib.DeviceLayer(L)
    x = torch.from_numpy(s.make_activations(1, L, 2)).cuda()
    none = lent("none")

    def microseconds(batch):
        y = torch.empty((batch, out), dtype=torch.float16, device="cuda")
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(50):
            gpu_lib.gemv(dl, x[:batch], out=y, workspace=none)
        end.record()
        torch.cuda.synchronize()
        return begin.elapsed_time(end) * 20.0
    microseconds(1), microseconds(2)
    times = sorted((microseconds(1), microseconds(2)) for _ in range(7))
    one, two = sorted(t[0] for t in times)[3], sorted(t[1] for t in times)[3]
    assert one <= 1.1 * two, "one row %.1f us, two rows %.1f us" % (one, two)
