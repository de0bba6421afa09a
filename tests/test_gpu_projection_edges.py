"""GPU parity of the router projection (and of the scores fused behind it) where its kernels change hands or have remainders:
rows and columns around the 32 x 32 tiles, reduction lengths around a matrix instruction, misaligned rows, and the token
counts at which bf16 leaves the split kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_12801_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,d,E", [
    (1, 1, 1), (31, 7, 33), (32, 8, 32), (33, 15, 31), (64, 16, 64), (65, 17, 65), (40, 64, 96), (95, 40, 97), (70, 1000, 127),
    (129, 136, 128), (33, 2056, 129), (50, 72, 300), (8192, 64, 128), (8193, 64, 128), (16384, 64, 64), (16385, 64, 32), (16385, 40, 96),
    (8193, 33, 128), (8200, 50, 70), (8250, 34, 90), (8193, 100, 80), (4097, 48, 160), (16384, 64, 128), (16385, 64, 128), (8255, 37, 48),
    (8195, 20, 20), (8193, 31, 97), (77, 24, 8), (300, 34, 16), (16384, 16, 80), (16385, 16, 100), (16385, 16, 64), (100, 18, 66), (90, 20, 100),
])
def test_projection_edges(ms, T, d, E, dtype):
    print(f"projection edges T={T} d={d} E={E} {dtype}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + d + E)
    x = torch.randn(T, d, generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    W = torch.randn(d, E, generator=gen, device="cuda").to(x.dtype)
    b = torch.randn(E, generator=gen, device="cuda")
    L = ms.router_logits(x, W, b)
    xs, Ws, bs = x.double().cpu(), W.double().cpu(), b.double().cpu()
    ref, mag = xs @ Ws + bs, xs.abs() @ Ws.abs() + bs.abs()
    assert ((L.double().cpu() - ref).abs() <= 1e-6 * mag).all()
    k = min(3, E)
    both = ms.router_softtopk(x, W, b, k, t=1.0)
    scores, q = ms.softtopk(L, k, 1.0)
    assert torch.equal(both["logits"], L) and torch.equal(both["scores"], scores) and torch.equal(both["q"], q)


@pytest.mark.parametrize("dtype,xo,wo", [("bf16", 1, 0), ("bf16", 0, 1), ("bf16", 2, 2), ("bf16", 3, 3), ("fp32", 1, 1)])
@pytest.mark.parametrize("T,d,E", [(70, 64, 64), (40, 66, 128), (8200, 64, 32), (33, 40, 96)])
def test_operands_off_their_alignment(ms, T, d, E, dtype, xo, wo):
    print(f"projection operands T={T} d={d} E={E} {dtype} {xo} {wo}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(T + d + E)
    x = torch.randn(T * d + 8, generator=gen, device="cuda").to(dt)[xo:xo + T * d].view(T, d)
    W = torch.randn(d * E + 8, generator=gen, device="cuda").to(dt)[wo:wo + d * E].view(d, E)
    L = ms.router_logits(x, W, None)
    xs, Ws = x.double().cpu(), W.double().cpu()
    assert ((L.double().cpu() - xs @ Ws).abs() <= 1e-6 * (xs.abs() @ Ws.abs())).all()
    both = ms.router_softtopk(x, W, None, 3, t=1.0)
    scores, q = ms.softtopk(L, 3, 1.0)
    assert torch.equal(both["logits"], L) and torch.equal(both["scores"], scores) and torch.equal(both["q"], q)


@pytest.mark.parametrize("T,d,E", [(8192, 24, 256), (8193, 24, 256), (12288, 20, 160), (12289, 24, 132), (16384, 24, 100), (16385, 24, 128),
                                   (24576, 16, 96), (24577, 20, 66), (20011, 24, 78), (40000, 8, 128)])
def test_fp32_rows_do_not_depend_on_their_number(ms, T, d, E):
    """Workgroups of 32 and of 64 rows add up the same parts in the same order: the ends of a batch and what is beyond a workgroup's
    rows have to agree with the same rows in batches of one workgroup each."""
    print(f"projection rows T={T} d={d} E={E}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + d + E)
    x = torch.randn(T, d, generator=gen, device="cuda")
    W = torch.randn(d, E, generator=gen, device="cuda")
    out = ms.router_softtopk(x, W, None, 3, t=1.0)
    assert torch.equal(out["logits"], ms.router_logits(x, W, None))
    for a in (0, 32, 8160, T // 64 * 32, (T - 1) // 64 * 64, (T - 1) // 32 * 32, T - 32):
        assert torch.equal(out["logits"][a:a + 32], ms.router_logits(x[a:a + 32].contiguous(), W, None)), a


@pytest.mark.parametrize("T,d,E,k,bias", [
    (8193, 64, 256, 8, True), (8250, 128, 129, 3, False), (8255, 192, 160, 8, True), (9000, 256, 132, 1, True), (16384, 64, 256, 8, False),
    (16383, 320, 255, 5, True), (16385, 64, 256, 8, True), (28608, 64, 130, 2, True), (28609, 64, 130, 2, True), (28673, 448, 224, 8, True),
    (8200, 512, 193, 64, True), (8200, 576, 256, 33, False), (8222, 768, 161, 4, True)])
def test_whole_rows_of_more_than_128_experts(ms, T, d, E, k, bias):
    """129 to 256 experts in one workgroup (8193 to 16384 tokens, and where sets of 256 workgroups are nearly full): the same bits as the
    projection kernel and the score kernel behind it, with one to twelve slabs of d, a last workgroup of few rows and a last block of
    few columns."""
    print(f"whole rows T={T} d={d} E={E} k={k}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T + d + E)
    x = torch.randn(T, d, generator=gen, device="cuda").to(torch.bfloat16)
    W = (torch.randn(d, E, generator=gen, device="cuda") / d ** 0.5).to(torch.bfloat16)
    W[:, E - 1] *= 3.0                       # (the column that stands in for those beyond the last one is a large one)
    b = torch.randn(E, generator=gen, device="cuda") if bias else None
    out = ms.router_softtopk(x, W, b, k, 1.0)
    L = ms.router_logits(x, W, b)
    scores, q = ms.softtopk(L, k, 1.0)
    assert torch.equal(out["logits"], L) and torch.equal(out["scores"], scores) and torch.equal(out["q"], q)
    rows = slice(T - 70, T)
    ref, mag = x[rows].double().cpu() @ W.double().cpu(), x[rows].double().cpu().abs() @ W.double().cpu().abs()
    if bias:
        ref, mag = ref + b.double().cpu(), mag + b.double().cpu().abs()
    assert ((L[rows].double().cpu() - ref).abs() <= 1e-6 * mag).all()
    with pytest.raises(ms.MaxScoreError):
        ms.router_softtopk(x, W, b, k, 1.0, want_logits=False)
