"""Multi-dot and update on both sides of the lines of their launch shapes.

Tiles per format (4096 rows for the 8- and 16-bit formats, 2048 for the
others): 512 (whole vectors, full ring), 768 (three blocks per CU), 769 and
1000 with a ragged last tile (two blocks per CU by LDS padding; none for
e4m3).  Against float64 products of the decoded vectors on the GPU: |err| <=
2 * 4 n 2^-53 sum |v w| for the dots, both sides' sums counted, and
8 (j + 1) 2^-53 (|w| + sum |h v|) for the update.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["fp64", "fp32", "fp16", "e4m3"])
@pytest.mark.parametrize("tiles,cut", [(512, 0), (768, 0), (769, 1), (1000, 37)])
@pytest.mark.parametrize("j", [1, 9])
def test_full_grids(fmt, tiles, cut, j):
    import paper_2009_12101_amd as cbg
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    n = tiles * (2048 if fmt in ("fp64", "fp32") else 4096) - cut
    print(f"multidot grid {fmt} n={n} j={j}", flush=True)
    gen = torch.Generator(device=dev).manual_seed(n + j)
    ld = cbg.basis_ld(n)
    by = cbg.FORMAT_BYTES[fmt]
    V = torch.zeros((j, ld * by), dtype=torch.uint8, device=dev)
    dec = torch.empty((j, n), dtype=torch.float64, device=dev)
    scales = torch.empty(j, dtype=torch.float64, device=dev)
    for k in range(j):
        v = torch.randn(n, dtype=torch.float64, device=dev, generator=gen) / n ** 0.5
        q, s = cbg.encode(fmt, v)
        V[k, :n * by] = q.view(torch.uint8)[:n * by]
        scales[k] = s[0]
        dec[k] = cbg.decode(fmt, q, s, n)
    w = torch.randn(n, dtype=torch.float64, device=dev, generator=gen)
    h = cbg.multidot(fmt, V.view(-1), ld, scales, n, j, w)
    ref = (dec * w).sum(dim=1)
    assert torch.all((h - ref).abs() <= 8 * n * 2.0 ** -53 * (dec * w).abs().sum(dim=1))
    w2 = w.clone()
    norms = cbg.update(fmt, V.view(-1), ld, scales, n, j, h, w2)
    bound = 8 * (j + 1) * 2.0 ** -53 * (w.abs() + (h.abs()[:, None] * dec.abs()).sum(dim=0))
    assert torch.all((w2 - (w - (h[:, None] * dec).sum(dim=0))).abs() <= bound)
    two = torch.linalg.vector_norm(w2)
    assert (norms[0] - two).abs() <= 2 * n * 2.0 ** -53 * two
    assert norms[1] == w2.abs().max()
