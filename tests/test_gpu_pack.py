"""The packed layout of the header and its column sums, byte for byte, at the edges of the pack kernel's blocks
(512 bytes of K per block, 1 KiB blocks for columns of up to 2 KiB), of the 16-byte chunks and of the panels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def layout(B, shift):
    """Packed bytes and column sums from the header's definition."""
    N, K = B.shape
    Np = -(-N // 32) * 32
    if B.dtype == np.int16:
        Ke = -(-K // 32) * 32
        hi, lo = np.zeros((Np, Ke), np.int64), np.zeros((Np, Ke), np.int64)
        b = B.astype(np.int64)
        hi[:N, :K], lo[:N, :K] = b >> 8, (b & 255) - 128
        rows = np.stack([hi.reshape(Np, -1, 32), lo.reshape(Np, -1, 32)], axis=2).reshape(Np, 2 * Ke)
        sums = np.zeros(Np, np.int64)
        sums[:N] = (b - 128).sum(axis=1)
    else:
        rows = np.zeros((Np, -(-K // 64) * 64), np.int64)
        rows[:N, :K] = B.astype(np.int64) - shift
        sums = rows.sum(axis=1)
    frag = rows.astype(np.int8).reshape(Np // 32, 32, -1, 2, 16).transpose(0, 2, 3, 1, 4)
    return np.concatenate([frag.reshape(-1).view(np.uint8), sums.astype(np.int32).view(np.uint8)])


@pytest.mark.parametrize("kind", ["s8", "u8", "s16"])
@pytest.mark.parametrize("K", [1, 3, 6, 13, 64, 500, 511, 1023, 1024, 1030, 2047, 2048, 2049, 2570])
def test_pack_layout(kind, K):
    import torch
    import paper_1910_00178_amd as ng
    ctx = ng.ngemm_create(0)
    rng = np.random.default_rng(K)
    dt = {"s8": np.int8, "u8": np.uint8, "s16": np.int16}[kind]
    info = np.iinfo(dt)
    size = ng.ngemm_packed_b_bytes_s16 if kind == "s16" else ng.ngemm_packed_b_bytes
    pack = {"s8": ng.ngemm_pack_b, "u8": ng.ngemm_pack_b_u8, "s16": ng.ngemm_pack_b_s16}[kind]
    for N, gap in ((1, 0), (32, 3), (45, 0), (70, 1)):
        B = rng.integers(info.min, info.max + 1, size=(N, K + gap)).astype(dt)
        dev = torch.from_numpy(B).cuda()
        n = size(K, N)
        packed = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
        h = pack(ctx, K, N, dev, K + gap, packed, n)
        got = packed.cpu().numpy()
        ng.ngemm_packed_b_free(h)
        assert np.array_equal(got[:n], layout(B[:, :K], 128 if kind == "u8" else 0)), (N, gap)
        assert (got[n:] == 0xA5).all(), "written past the packed buffer"
    ng.ngemm_destroy(ctx)


def test_widest_operand():
    """2^28 columns and more: as many panels as workgroups of 512 threads would need 2^32 threads for, and packed bytes far beyond
    4 GiB.  Columns on both sides of that mark against the header's definition."""
    import torch
    import paper_1910_00178_amd as ng
    N, K = (1 << 28) + 7, 3
    ctx = ng.ngemm_create(0)
    B = torch.randint(-128, 128, (N, K), dtype=torch.int8, device="cuda")
    n = ng.ngemm_packed_b_bytes(K, N)
    packed = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")
    h = ng.ngemm_pack_b(ctx, K, N, B, K, packed, n)
    torch.cuda.synchronize()
    ng.ngemm_packed_b_free(h)
    Np = -(-N // 32) * 32
    for first in (0, 1 << 26, (1 << 28) - 32, 1 << 28):          # a panel of 32 columns: two fragments of 1 KiB
        cols = B[first:first + 32].cpu().numpy()
        want = layout(cols, 0)
        assert np.array_equal(packed[first * 64:first * 64 + 2048].cpu().numpy(), want[:2048]), first
        at = Np * 64 + 4 * first
        assert np.array_equal(packed[at:at + 128].cpu().numpy(), want[2048:]), first
    ng.ngemm_destroy(ctx)
