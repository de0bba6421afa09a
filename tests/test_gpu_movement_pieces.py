"""GPU: rows whose length ends within a piece of the combine kernel, and sizes on both sides of the lines beyond which rows pass the
caches, against plain indexing (the rows out are a copy: exact; the rows back against 64 bits)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _case(T, d, E, k, C, dtype):
    """An assignment with empty slots and places beyond the buffers, made without the library."""
    gen = torch.Generator(device="cuda").manual_seed(T + d + k)
    assign = torch.rand(T, E, generator=gen, device="cuda").topk(k, dim=1).indices.int()
    assign[torch.rand(T, k, generator=gen, device="cuda") < 0.1] = -1
    pos = torch.randint(0, C + 1, (T, k), generator=gen, device="cuda", dtype=torch.int32)
    gates = torch.rand(T, k, generator=gen, device="cuda")
    buf = torch.randn(E, C, d, generator=gen, device="cuda").to(dtype)
    return assign, pos, gates, buf


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("T,d,E,k,C", [
    (70, 8, 4, 1, 9), (70, 256, 4, 2, 9), (70, 264, 4, 2, 9), (70, 504, 5, 3, 9), (70, 512, 4, 1, 9), (70, 520, 6, 5, 9), (70, 776, 4, 2, 9),
    (70, 1016, 9, 8, 9), (70, 1288, 9, 7, 9), (70, 64, 9, 4, 9), (70, 200, 9, 8, 9), (70, 256, 9, 5, 9), (8200, 256, 64, 8, 1030),
    (3000, 1288, 16, 5, 900),           # two pieces to a wavefront
    (8200, 1800, 16, 4, 2050),          # past the caches, loads ahead
    (8200, 3080, 16, 2, 1025),          # ... one after the other
])
def test_combine_ends_of_rows(T, d, E, k, C, dtype):
    import paper_2508_12801_amd as ms
    print(f"combine ends of rows T={T} d={d} E={E} k={k} C={C} {dtype}", flush=True)
    assign, pos, gates, buf = _case(T, d, E, k, C, torch.bfloat16 if dtype == "bf16" else torch.float32)
    y = ms.combine(buf, assign, pos, gates)
    ref, size = torch.zeros(T, d, dtype=torch.float64, device="cuda"), torch.zeros(T, d, dtype=torch.float64, device="cuda")
    for s in range(k):
        ok = (assign[:, s] >= 0) & (pos[:, s] < C)
        rows = buf[assign[:, s].clamp(min=0).long(), pos[:, s].clamp(max=C - 1).long()].double() * gates[:, s].double()[:, None]
        rows = torch.where(ok[:, None], rows, torch.zeros_like(rows))
        ref += rows
        size += rows.abs()
    # k fused multiply-adds in fp32: 2^-24 each, of no more than the sum of the terms' sizes
    assert ((y.double() - ref).abs() <= (k + 1) * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("T,d,E,k,C,dtype", [
    (4100, 264, 8, 2, 1030, "bf16"),
    (22000, 1544, 16, 2, 2800, "bf16"),  # x, buffers and results 324 MiB
    (24001, 1544, 16, 2, 3050, "bf16"),  # ... 353 MiB, buffers 144
    (9001, 2056, 16, 3, 1700, "fp32"),   # ... 354 MiB, buffers 213
    (13001, 2056, 16, 3, 1700, "fp32"),  # rows of 102 MiB, read past them as well
])
def test_rows_out_either_side_of_the_caches(T, d, E, k, C, dtype):
    import paper_2508_12801_amd as ms
    print(f"rows out T={T} d={d} E={E} k={k} C={C} {dtype}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn(T, d, generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    # every expert's list holds ascending tokens, as many as it has places or fewer
    lists = [torch.randperm(T, generator=gen, device="cuda")[:C - 7 * e].sort().values for e in range(E)]
    offsets = torch.tensor([0] + [len(t) for t in lists], device="cuda").cumsum(0).int()
    out = ms.dispatch_tokens(x, offsets, torch.cat(lists).int(), E, C)
    for e, t in enumerate(lists):
        assert torch.equal(out[e, :len(t)], x[t]) and not out[e, len(t):].any()
