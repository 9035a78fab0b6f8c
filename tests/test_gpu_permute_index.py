"""The permutes find token and slab of an element by multiplication: odd divisors, at the largest index 32 bits are used for."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,D,P,many", [
    (102261000, 3, 7, 3, False),   # one byte per vector: 2 147 481 000 vectors, a row of 21, runs of 7
    (30011, 24, 80, 3, True),      # 16-byte vectors: rows of 480, 320 and 60, runs of 160 and 20
    (4099, 15, 48, 5, True),
    (1, 7, 16, 7, True),
])
def test_odd_rows_and_runs(T, H, D, P, many):
    import torch
    from paper_2412_01523_amd import binding as fx
    print(f"permute index: T={T} H={H} D={D} P={P}", flush=True)
    ctx = fx.Context(0)
    heads = [H] if not many else [H, P, 2 * P]
    xs = [torch.empty((T, h, D), dtype=torch.uint8 if not many else torch.int32, device="cuda") for h in heads]
    for x in xs:
        flat = x.view(-1)
        for i in range(0, flat.numel(), 1 << 28):  # (filled piece by piece: the index array would be 16 GB)
            n = min(1 << 28, flat.numel() - i)
            flat[i:i + n] = (torch.arange(i, i + n, device="cuda") * 2654435761 >> 13).to(x.dtype)
    ys = [torch.empty((P, T, h // P, D), dtype=x.dtype, device="cuda") for x, h in zip(xs, heads)]
    if many:
        fx.flexsp_pack_many(ctx, xs, ys, P)
    else:
        fx.flexsp_pack(ctx, xs[0], ys[0], P)
    for x, y, h in zip(xs, ys, heads):
        for r in range(P):
            assert torch.equal(y[r], x[:, r * (h // P):(r + 1) * (h // P)])
    zs = [torch.zeros_like(x) for x in xs]
    if many:
        fx.flexsp_unpack_many(ctx, ys, zs)
    else:
        fx.flexsp_unpack(ctx, ys[0], zs[0])
    for x, z in zip(xs, zs):
        assert torch.equal(x, z)
    ctx.close()
