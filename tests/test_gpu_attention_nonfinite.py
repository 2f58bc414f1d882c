"""Infinities and NaN in the paged cache of a ragged decode attention (bf16 caches on matrix cores, whose
queries and probabilities are sums of bf16 planes): a row sees those of its own keys only, and sees them
as plain arithmetic does. An infinite value makes its dim infinite, an infinite key gives its query NaN or,
at minus infinity, weight zero, a NaN key spoils the rows that attend it, and nothing past a row's last key
reaches the row. Against numpy in 64 bits; finite results to relative 1e-4 of the row, as the finite cases
of the same call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _reference(q, k, v):
    """One query over its keys, in 64 bits."""
    with np.errstate(all="ignore"):
        s = k @ q / np.sqrt(len(q))
        p = np.exp(s - s.max())
        return (p[:, None] * v).sum(0) / p.sum()


@pytest.mark.parametrize("keys,chunk", [(40, 64), (130, 64), (163, 48)])
@pytest.mark.parametrize("hq,hkv,dh", [(8, 2, 128), (8, 1, 64), (2, 2, 64)])
def test_rows_see_their_own_nonfinite_keys(hq, hkv, dh, keys, chunk):
    _rows_see_their_own(hq, hkv, dh, keys, chunk, torch.bfloat16)


@pytest.mark.parametrize("keys,chunk", [(40, 64), (130, 64), (163, 48)])
@pytest.mark.parametrize("hq,hkv,dh", [(8, 2, 128), (8, 1, 64)])
def test_rows_of_fp32_caches_do(hq, hkv, dh, keys, chunk):
    """The one-row split of fp32 caches, whose waves may hold a single key: a wave of nothing but NaN scores, or of
    nothing but minus infinity, counts as such."""
    _rows_see_their_own(hq, hkv, dh, keys, chunk, torch.float32)


def _rows_see_their_own(hq, hkv, dh, keys, chunk, dtype):
    from paper_2605_30852_amd import binding as B
    rows, G, inf = 4, hq // hkv, float("inf")
    rng = np.random.default_rng(keys + dh)
    lens = np.array([keys - i for i in range(rows)], dtype=np.int32)
    pages = (keys + 15) // 16 + 1
    base = torch.from_numpy(rng.standard_normal((2, pages * 16, hkv, dh)).astype(np.float32)).to(dtype)
    q = rng.standard_normal((rows, hq, dh)).astype(np.float32)
    table = rng.permutation(pages).astype(np.int32)
    marks = {"value of the longest row's last key": [(1, keys - 1, 0, 3, inf)],
             "value of every row": [(1, 7, hkv - 1, 5, -inf)],
             "key of every row": [(0, 9, 0, 0, inf)],
             "NaN key of two rows": [(0, keys - 2, 0, 1, float("nan"))],
             "key of the longest row at minus infinity": [(0, keys - 1, 0, 0, -inf)],
             "past every row": [(0, keys, 0, 2, float("nan")), (1, keys, 0, 2, inf)]}
    for what, at in marks.items():
        kv = base.clone()
        for part, key, head, dim, x in at:
            kv[part, key, head, dim] = x
        pool = torch.empty(pages, 2, hkv, 16, dh, dtype=dtype)
        pool[torch.from_numpy(table).long()] = kv.view(2, pages, 16, hkv, dh).permute(1, 0, 3, 2, 4)
        pool_d, q_d, table_d = pool.cuda(), torch.from_numpy(q).cuda(), torch.from_numpy(table).cuda()
        out = torch.zeros(rows, hq, dh, device="cuda")
        nb = B.decode_attention_workspace_bytes(rows, hkv, dh, lens, chunk)
        ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")
        print(f"[{what}: {hq}/{hkv}x{dh} keys {keys} chunk {chunk}]", flush=True)
        B.spd_decode_attention(q_d.data_ptr(), pool_d.data_ptr(), table_d.data_ptr(), pages, lens, hq, hkv, dh,
                               B.SPD_BF16 if dtype == torch.bfloat16 else B.SPD_F32, chunk, out.data_ptr(),
                               (ws.data_ptr() + 255) // 256 * 256, nb, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got, x = out.cpu().numpy(), kv.double().numpy()
        for i in range(rows):
            for h in range(hq):
                n = int(lens[i])
                want = _reference(q[i, h].astype(np.float64), x[0, :n, h // G], x[1, :n, h // G])
                fin = np.isfinite(want)
                assert np.array_equal(got[i, h][~fin], want[~fin], equal_nan=True), (what, i, h)
                err = np.linalg.norm((got[i, h] - want)[fin])
                assert err <= 1e-4 * max(np.linalg.norm(want[fin]), 1e-30), (what, i, h, err)


def _call_us(B, args, n=5):
    """Best time of n calls, in microseconds."""
    best = float("inf")
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        B.spd_decode_attention(*args, torch.cuda.current_stream().cuda_stream)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("what", ["NaN query", "NaN key", "infinite value", "key at minus infinity"])
def test_long_split_with_nonfinite_stays_bounded(what):
    """One split of 8192 keys whose every query needs the plain form: right, and within 100 times the finite
    call. 16 queries in turn, each two passes of 32 keys a thread, are some 130000 dependent steps; a form in
    which every thread walks all keys twice for each of its dim pairs needs 4.2 million a query."""
    from paper_2605_30852_amd import binding as B
    rows, hq, hkv, dh, keys = 4, 4, 1, 128, 8192
    rng = np.random.default_rng(11)
    lens = np.array([keys - i for i in range(rows)], dtype=np.int32)
    pages = keys // 16
    kv = torch.from_numpy(rng.standard_normal((pages, 2, hkv, 16, dh)).astype(np.float32)).bfloat16()
    q = torch.from_numpy(rng.standard_normal((rows, hq, dh)).astype(np.float32))
    table = torch.arange(pages, dtype=torch.int32).cuda()
    nb = B.decode_attention_workspace_bytes(rows, hkv, dh, lens, keys)
    ws = torch.empty(nb + 256, dtype=torch.uint8, device="cuda")
    out = torch.zeros(rows, hq, dh, device="cuda")

    def args(pool, qd):
        return (qd.data_ptr(), pool.data_ptr(), table.data_ptr(), pages, lens, hq, hkv, dh, B.SPD_BF16, keys,
                out.data_ptr(), (ws.data_ptr() + 255) // 256 * 256, nb)
    pool, qd = kv.cuda(), q.cuda()
    print(f"[{what}: finite]", flush=True)
    finite = _call_us(B, args(pool, qd))
    if what == "NaN query":
        q[:, :, 5] = float("nan")
    elif what == "NaN key":
        kv[3, 0, 0, 2, 7] = float("nan")
    elif what == "infinite value":
        kv[3, 1, 0, 2, 7] = float("inf")
    else:
        q[:, :, 7] = q[:, :, 7].abs() + 0.1
        kv[3, 0, 0, 2, 7] = -float("inf")
    pool, qd = kv.cuda(), q.cuda()
    print(f"[{what}]", flush=True)
    took = _call_us(B, args(pool, qd))
    got, x = out.cpu().numpy(), kv.double().numpy()
    k, v = (x[:, p].transpose(0, 2, 1, 3).reshape(-1, hkv, dh) for p in (0, 1))
    for i in range(rows):
        for h in range(hq):
            n = int(lens[i])
            want = _reference(q[i, h].double().numpy(), k[:n, 0], v[:n, 0])
            fin = np.isfinite(want)
            assert np.array_equal(got[i, h][~fin], want[~fin], equal_nan=True), (i, h)
            assert np.linalg.norm(got[i, h][fin] - want[fin]) <= 1e-4 * max(np.linalg.norm(want[fin]), 1e-30), (i, h)
    print(f"  finite {finite:.1f} us, {what} {took:.1f} us", flush=True)
    assert took <= 100 * finite, (finite, took)
