"""GPU parity of the token-block dispatch and of the chunked combine where they can go wrong: token counts around the block
sizes, row lengths around the chunks of a wavefront, lists that are not in token order, tokens in more lists than a block
keeps, entries outside the batch, slots that are empty or outside the buffers."""
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


@pytest.mark.parametrize("T,E,C,lists", [
    (4095, 5, 900, "sorted"), (4096, 5, 900, "sorted"), (4099, 300, 20, "sorted"), (8193, 17, 800, "shuffled"),
    (16385, 40, 900, "sorted"), (16384, 24, 700, "crowded"), (32771, 3, 9000, "outside"), (32768, 600, 70, "sorted"),
])
def test_dispatch_blocks(ms, T, E, C, lists):
    print(f"dispatch blocks T={T} E={E} C={C} {lists}", flush=True)
    rng = np.random.default_rng(T + E)
    d = 8 if E > 100 else 24
    x = torch.from_numpy(rng.integers(1, 1 << 30, (T, d)).astype(np.int32)).cuda().view(torch.float32)
    segs = []
    for e in range(E):
        n = int(rng.integers(0, C + 1)) if e % 3 else (0 if e % 2 else C)
        t = np.sort(rng.choice(T, n, replace=False))
        if lists == "shuffled" and e % 4 == 1:
            rng.shuffle(t)
        if lists == "crowded" and n:
            t[:min(n, 40)] = np.sort(rng.integers(100, 103, min(n, 40)))
            t = np.sort(t)
        if lists == "outside" and n:
            t[-1], t[0] = T + 1, -3
        segs.append(t)
    off = np.concatenate([[0], np.cumsum([len(s) for s in segs])]).astype(np.int32)
    tok = np.concatenate(segs).astype(np.int32)
    buf = ms.dispatch_tokens(x, torch.from_numpy(off).cuda(), torch.from_numpy(tok).cuda(), E, C).view(torch.int32)
    rows = torch.from_numpy(np.where((tok >= 0) & (tok < T), tok, 0).astype(np.int64)).cuda()
    for e in range(E):
        n = int(off[e + 1] - off[e])
        assert torch.equal(buf[e, :n], x.view(torch.int32)[rows[off[e]:off[e + 1]]]), e
        assert not buf[e, n:].any(), e


@pytest.mark.parametrize("d,k,dtype", [(8, 1, "bf16"), (512, 2, "bf16"), (520, 9, "bf16"), (1032, 8, "bf16"), (2048, 3, "bf16"),
                                       (2056, 5, "bf16"), (4104, 2, "bf16"), (4, 64, "fp32"), (256, 7, "fp32"), (2052, 3, "fp32")])
def test_combine_chunks(ms, d, k, dtype):
    print(f"combine chunks d={d} k={k} {dtype}", flush=True)
    rng = np.random.default_rng(d + k)
    T, E, C = 37, k + 3, 11
    buf = torch.from_numpy(rng.standard_normal((E, C, d), dtype=np.float32)).cuda()
    buf = buf.to(torch.bfloat16) if dtype == "bf16" else buf
    a = np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)
    pos = rng.integers(0, C, (T, k)).astype(np.int32)
    g = rng.random((T, k), dtype=np.float32)
    a[3], a[5, -1], pos[7, 0] = -1, E, C                      # an empty row, an expert and a place that do not exist
    y = ms.combine(buf, torch.from_numpy(a).cuda(), torch.from_numpy(pos).cuda(), torch.from_numpy(g).cuda()).cpu().numpy()
    ok = (a >= 0) & (a < E) & (pos < C)
    rows = buf.float().cpu().numpy().astype(np.float64)[np.where(ok, a, 0), np.where(ok, pos, 0)]
    terms = rows * (g.astype(np.float64) * ok)[:, :, None]
    assert (np.abs(y - terms.sum(axis=1)) <= 1e-6 * np.abs(terms).sum(axis=1) + 1e-30).all()


@pytest.mark.parametrize("T,d,E,C", [(4096, 8, 1, 7), (4096, 8, 3, 21), (5000, 8, 7, 1031), (4099, 8, 5, 70001), (10000, 8, 64, 172),
                                     (4096, 8, 1024, 513), (16384, 8192, 3, 9001)])
def test_rows_without_a_token(ms, T, d, E, C):
    """The rows behind every list's end are zeros: fewer rows than a workgroup looks at, more than all of them look at in one turn, and
    buffers and tokens beyond the last cache (workgroups of sixteen wavefronts)."""
    print(f"rows without a token T={T} d={d} E={E} C={C}", flush=True)
    rng = np.random.default_rng(T + C)
    x = torch.randint(1, 1 << 15, (T, d), dtype=torch.int16, device="cuda").view(torch.bfloat16)
    n = np.minimum(rng.integers(0, C + 1, E), T)
    n[0] = min(C, T)
    tok = np.concatenate([np.sort(rng.choice(T, c, replace=False)) for c in n]).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    buf = torch.full((E, C, d), -1, dtype=torch.int16, device="cuda").view(torch.bfloat16)
    ms.dispatch_tokens(x, torch.from_numpy(off).cuda(), torch.from_numpy(tok).cuda(), E, C, out=buf)
    rows = torch.from_numpy(tok.astype(np.int64)).cuda()
    for e in range(E):
        assert torch.equal(buf.view(torch.int16)[e, :n[e]], x.view(torch.int16)[rows[off[e]:off[e + 1]]]), e
        assert not buf.view(torch.int16)[e, n[e]:].any(), e


@pytest.mark.parametrize("d,k,dtype", [(520, 3, "bf16"), (1024, 4, "bf16"), (1032, 5, "bf16"), (1544, 9, "bf16"), (2048, 8, "bf16"),
                                       (260, 4, "fp32"), (1000, 6, "fp32"), (4100, 64, "fp32")])
def test_combine_two_pieces(ms, d, k, dtype):
    """Buffers of at least 24 MiB, and tokens for 2560 wavefronts, take two kilobytes of a row to a wavefront: the same sums in the same
    order as from buffers just large enough for the rows."""
    print(f"combine two pieces d={d} k={k} {dtype}", flush=True)
    rng = np.random.default_rng(d + k)
    T, E, C = 2563 if k < 16 else 641, k + 2, 7
    far = (24 << 20) // (E * d * (2 if dtype == "bf16" else 4)) + 1
    small = torch.from_numpy(rng.standard_normal((E, C, d), dtype=np.float32)).cuda()
    small = small.to(torch.bfloat16) if dtype == "bf16" else small
    large = torch.zeros(E, far, d, dtype=small.dtype, device="cuda")
    places = torch.from_numpy(np.sort(rng.choice(far, C, replace=False))).cuda()
    large[:, places] = small
    a = torch.from_numpy(np.argsort(rng.random((T, E)), axis=1)[:, :k].astype(np.int32)).cuda()
    a[3], a[5, -1] = -1, E
    pos = torch.from_numpy(rng.integers(0, C, (T, k))).cuda()
    g = torch.from_numpy(rng.random((T, k), dtype=np.float32)).cuda()
    y = ms.combine(large, a, places[pos].int(), g)
    assert torch.equal(y, ms.combine(small, a, pos.int(), g))
    ok = (a >= 0) & (a < E)
    terms = small.double()[torch.where(ok, a, 0).long(), pos] * (g.double() * ok)[:, :, None]
    assert ((y - terms.sum(dim=1)).abs() <= 1e-6 * terms.abs().sum(dim=1) + 1e-30).all()


@pytest.mark.parametrize("T,d,E,k,C,dtype", [
    (1, 8, 4, 3, 2, "bf16"), (5, 520, 3, 3, 6, "bf16"), (70, 504, 8, 4, 40, "fp32"), (33, 1032, 6, 5, 30, "bf16"), (257, 512, 16, 8, 130, "bf16"),
    (65, 64, 16, 9, 50, "bf16"), (2600, 1016, 8, 6, 2000, "bf16"), (2570, 1032, 8, 4, 1300, "fp32"), (2561, 2040, 4, 3, 2000, "bf16"),
    (40, 72, 4, 2, 30, "bf16"), (40, 72, 4, 1, 30, "fp32")])
def test_combine_with_slots_read_ahead(ms, T, d, E, k, C, dtype):
    """Slots that are empty (the first, the last, all of a token's) and lanes beyond a row add nothing, whatever they read: the first row of
    the buffer and every place that nothing points to hold NaN."""
    print(f"combine read ahead T={T} d={d} E={E} k={k} C={C} {dtype}", flush=True)
    rng = np.random.default_rng(T + d + k)
    places = 1 + rng.permutation(E * C - 1)                  # (place 0 stays unused)
    keep = rng.random((T, k)) < 0.7
    keep[0, 0] = False
    keep[T // 2] = False
    keep[T - 1, k - 1] = False
    n = int(keep.sum())
    assert n <= len(places)
    at = np.full((T, k), -1, np.int64)
    at[keep] = places[:n]
    a = np.where(keep, at // C, -1).astype(np.int32)
    pos = np.where(keep, at % C, 0).astype(np.int32)
    g = rng.random((T, k)).astype(np.float32)
    buf = torch.full((E * C, d), float("nan"), device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
    rows = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32)).cuda().to(buf.dtype)
    buf[torch.from_numpy(at[keep]).cuda()] = rows
    y = ms.combine(buf.view(E, C, d), torch.from_numpy(a).cuda(), torch.from_numpy(pos).cuda(), torch.from_numpy(g).cuda()).cpu().numpy()
    terms = np.zeros((T, k, d))
    terms[keep] = rows.double().cpu().numpy() * g.astype(np.float64)[keep][:, None]
    # k fused multiply-adds in fp32: each rounds a partial sum once
    assert (np.abs(y - terms.sum(1)) <= k * 2.0 ** -24 * np.abs(terms).sum(1)).all()
