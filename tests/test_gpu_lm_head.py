"""GPU parity of the final RMSNorm + fp16 LM head against the fp64 reference
checker: full outputs on small shapes (ragged M, vocabulary not a multiple of
a workgroup's 128 rows) and sampled vocabulary rows at the 80-layer
configuration's full size (M = 64, H = 8192, V = 128256), tolerance
|gpu - ref| <= 2e-3 + 1e-2 |ref|."""
import numpy as np
import pytest

import gen
import oracle
from gen.workloads import CONFIGS, make_final_norm, make_lm_head

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2506_11309_amd as ss
    ss.lib()
    torch.cuda.set_device(0)


import paper_2506_11309_amd as ss  # noqa: E402
from gpu_helpers import check_close, dev, down16, up  # noqa: E402


def _run(h, gamma, W):
    M, H = h.shape
    V = W.shape[0]
    logits = torch.zeros((M, V), dtype=torch.int16, device=dev())
    ws = ss.workspace(ss.lm_head_workspace_bytes(M, H, V), dev())
    ss.lm_head(up(h), up(gamma), up(W), logits, ws)
    torch.cuda.synchronize()
    return down16(logits)


@pytest.mark.parametrize("M,H,V", [(1, 256, 16), (13, 512, 320), (32, 1024, 1040), (64, 384, 272)])
def test_lm_head_small_shapes(M, H, V):
    h = gen.normal_f16(71, M, (M, H))
    gamma = gen.normal_f16(72, M, (H,), 1.0, 0.02)
    W = gen.normal_f16(73, M, (V, H), 0.0, 0.02)
    got = _run(h, gamma, W)
    ref = oracle.lm_head(h, gamma, W)
    err, rel = check_close(got, ref, f"lm_head M={M} H={H} V={V}")
    print(f"lm_head M={M} H={H} V={V}: max abs err {err:.3g}, max rel err (|r|>=0.2) {rel:.3g}")


@pytest.mark.parametrize("M,H,V", [(1, 128, 16), (48, 128, 16384), (17, 640, 16400), (64, 128, 66800), (33, 1152, 4112),
                                   (16, 128, 131056), (49, 256, 118016)])
def test_lm_head_row_blocks(M, H, V):
    """64, 128 and 256 vocabulary rows per workgroup (up to 16384 columns, up
    to 65536 or an uneven last round, whole rounds of 256 workgroups), the
    last workgroup partly or almost wholly past V, K shorter than the ring of
    stages, every number of M-tiles."""
    h = gen.normal_f16(74, M, (M, H))
    gamma = gen.normal_f16(75, M, (H,), 1.0, 0.02)
    W = gen.normal_f16(76, M, (V, H), 0.0, 0.02)
    check_close(_run(h, gamma, W), oracle.lm_head(h, gamma, W), f"lm_head M={M} H={H} V={V}")


def test_lm_head_full_size_sampled_rows():
    cfg = CONFIGS["c5"]
    H, V, M = cfg.shape.H, cfg.vocab, cfg.T
    h = gen.normal_f16(cfg.seeds()["activations"], 7, (M, H))
    gamma = make_final_norm(cfg)
    W = make_lm_head(cfg)
    got = _run(h, gamma, W)
    del W
    rng = np.random.default_rng(5)
    rows = np.concatenate([[0, 1, V - 129, V - 128, V - 1], rng.choice(V, 59, replace=False)])
    ref = oracle.lm_head(h, gamma, make_lm_head(cfg, rows))
    err, rel = check_close(got[:, rows], ref, "lm_head c5 sampled rows")
    print(f"lm_head c5 (64 x 8192 x 128256), {len(rows)} sampled rows: max abs err {err:.3g}, rel {rel:.3g}")
    assert np.isfinite(got.view(np.float16).astype(np.float32)).all()


def test_lm_head_rejects_bad_arguments():
    h = torch.zeros((4, 256), dtype=torch.int16, device=dev())
    g = torch.zeros((256,), dtype=torch.int16, device=dev())
    W = torch.zeros((24, 256), dtype=torch.int16, device=dev())
    out = torch.zeros((4, 24), dtype=torch.int16, device=dev())
    ws = ss.workspace(ss.lm_head_workspace_bytes(4, 256, 24), dev())
    with pytest.raises(RuntimeError):
        ss.lm_head(h, g, W, out, ws)  # V % 16 != 0
    with pytest.raises(RuntimeError):
        ss.lm_head(h, g, W[:16], out, ss.workspace(16, dev()))  # workspace too small


@pytest.mark.parametrize("M,H,V", [(64, 1 << 25, 32), (17, (1 << 26) + 128, 48)])
def test_lm_head_long_rows(M, H, V):
    """Rows of 64 MiB and more (64 rows reach 4 GiB): against float64 on the
    GPU, with hidden states that are zero but for 4096 columns spread over
    the rows (the norm's sum of squares and the products see those alone)."""
    g = torch.Generator(device=dev())
    g.manual_seed(H + M)
    cols = torch.arange(4096, device=dev()) * (H // 4096) + torch.randint(0, H // 4096, (4096,), generator=g, device=dev())
    h = torch.zeros((M, H), dtype=torch.float16, device=dev())
    hc = torch.randn((M, 4096), generator=g, device=dev()).half()
    h[:, cols] = hc
    gamma = torch.ones(H, dtype=torch.float16, device=dev())
    W = torch.empty((V, H), dtype=torch.float16, device=dev()).normal_(0.0, 0.02 * (4096.0 / H) ** 0.5, generator=g)
    out = torch.zeros((M, V), dtype=torch.float16, device=dev())
    ws = ss.workspace(ss.lm_head_workspace_bytes(M, H, V), dev())
    ss.lm_head(h, gamma, W, out, ws)
    torch.cuda.synchronize()
    x = hc.double()
    xn = (x / (x.pow(2).sum(1, keepdim=True) / H + 1e-5).sqrt()).half().double()
    ref = xn @ W[:, cols].double().T
    check_close(down16(out.view(torch.int16)), ref.cpu().numpy().astype(np.float16).view(np.uint16),
                f"lm_head M={M} H={H} V={V}")
