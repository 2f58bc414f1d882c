"""The ragged decode attention with lengths that differ widely, in any order: rows that end in another row's
first split, at a split's or tile's edge, or long before it, beside the longest. bf16 caches share key tiles
between rows (32 / G rows a workgroup), so a row's last key, its split records and the splits that it has no key
in are all a matter of the launch's row masks. Against 64 bits; fp32 sums of exact products reach some 3e-7, the
bound is 1e-5 relative per row and head. The fp32 cache takes the same cases."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENS = [[1, 2000, 17, 640], [3, 64, 65, 128, 129, 700, 1500, 1999], [1999, 1, 1, 1, 1, 1, 1, 33], [1, 1300], [32, 1, 31, 33, 2, 63]]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("hq,hkv,dh,chunk", [(8, 2, 128, 64), (16, 2, 64, 128), (2, 2, 64, 2048), (4, 2, 128, 48)])
def test_any_lengths(hq, hkv, dh, chunk, dtype):
    from paper_2605_30852_amd import binding as B
    G = hq // hkv
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for lens in LENS:
        g = torch.Generator().manual_seed(sum(lens) + dh)
        rows, pages = len(lens), (max(lens) + 15) // 16 + 1
        pool = torch.randn(pages, 2, hkv, 16, dh, generator=g).to(dt)
        q = 1.5 * torch.randn(rows, hq, dh, generator=g)
        table = torch.randperm(pages, generator=g).int()
        ln = np.array(lens, dtype=np.int32)
        nb = B.decode_attention_workspace_bytes(rows, hkv, dh, ln, chunk)
        ws = torch.full((nb + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        pool_d, q_d, table_d = pool.cuda(), q.cuda(), table.cuda()
        out = torch.full((rows, hq, dh), float("nan"), device="cuda")
        print(f"[{dtype} {hq}/{hkv}x{dh} chunk {chunk} lens {lens}]", flush=True)
        B.spd_decode_attention(q_d.data_ptr(), pool_d.data_ptr(), table_d.data_ptr(), pages, ln, hq, hkv, dh,
                               B.SPD_BF16 if dtype == "bf16" else B.SPD_F32, chunk, out.data_ptr(),
                               (ws.data_ptr() + 255) // 256 * 256, nb, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        kv = pool[table.long()].double().permute(1, 2, 0, 3, 4).reshape(2, hkv, -1, dh)
        got = out.cpu().double()
        for i, n in enumerate(lens):
            for h in range(hq):
                k, v = kv[0, h // G, :n], kv[1, h // G, :n]
                want = torch.softmax(k @ q[i, h].double() / dh ** 0.5, 0) @ v
                err = float((got[i, h] - want).norm() / want.norm())
                assert err <= 1e-5, (lens, i, h, err)
