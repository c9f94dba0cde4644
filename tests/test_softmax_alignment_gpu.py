"""IndexSoftmax on rows that start at every alignment: column counts around the bounds of each row layout, contiguous rows
(odd strides), a probability tensor that starts off a word, and untouched bytes around it; and rows whose groups of four columns
are whole; bit-compared with the oracle."""
import numpy as np
import pytest

from test_parity_gpu import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu

COLS = [1, 2, 3, 253, 254, 255, 257, 1021, 1023, 2045, 2046, 2047, 4093, 4095, 6001, 8191, 16381, 16382, 16383, 16387]


@pytest.mark.parametrize("shift", [0, 1, 2, 3], ids=lambda s: f"shift{s}")
@pytest.mark.parametrize("masked", [False, True], ids=["all", "causal"])
def test_rows_at_every_alignment_bit_exact(torch_mod, oracle, masked, shift):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    ia = binding.IntAttn(device=0)
    rng = np.random.default_rng(41 + shift)
    for cols in COLS:
        for c_int in (5203, 2**25 + 1):  # the top-byte index map, the fp64 one
            rpm = min(5, cols) if masked else 0
            rows = 2 * rpm if masked else 5
            a = rng.integers(-3 * c_int, 3 * c_int, size=(rows, cols), dtype=np.int64).astype(np.int32)
            want = oracle.index_softmax(a, c_int, rows_per_matrix=rpm, causal=masked)
            # logits that start on any of the four alignments a 16-byte load can meet
            src = torch.full((shift + rows * cols + 4,), 2**31 - 1, dtype=torch.int32, device="cuda")
            src[shift:shift + rows * cols] = torch.from_numpy(a).cuda().reshape(-1)
            dst = torch.full((shift + rows * cols + 8,), 7, dtype=torch.uint8, device="cuda")
            ia.index_softmax(src[shift:shift + rows * cols].view(rows, cols), c_int, causal=masked, rows_per_matrix=rpm,
                             out=dst[shift:shift + rows * cols].view(rows, cols))
            torch.cuda.synchronize()
            got = dst.cpu().numpy()
            assert int((got[shift:shift + rows * cols].reshape(rows, cols) != want).sum()) == 0, (cols, c_int)
            assert (got[:shift] == 7).all() and (got[shift + rows * cols:] == 7).all(), (cols, c_int)
    ia.close()


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "off a word"])
@pytest.mark.parametrize("cols", [4, 60, 252, 256, 260, 512, 1020, 1028, 2044, 2048, 2052, 4096, 4100, 8188, 8192, 8196, 16380, 16384, 16388])
def test_rows_of_whole_groups_bit_exact(torch_mod, oracle, cols, shift):  # noqa: F811
    from paper_2511_21513_amd import binding

    torch = torch_mod
    rng = np.random.default_rng(cols)
    ia = binding.IntAttn(device=0)
    for rows, c_int in ((1, 5203), (7, 5203), (7, 2**25 + 1)):
        a = rng.integers(-3 * c_int, 3 * c_int, size=(rows, cols), dtype=np.int64).astype(np.int32)
        a[-1, -1] = a.max() + 1  # a maximum in the last column
        want = oracle.index_softmax(a, c_int)
        dst = torch.full((shift + rows * (cols + 8),), 7, dtype=torch.uint8, device="cuda")
        view = dst[shift:].view(rows, cols + 8)[:, :cols]
        ia.index_softmax(torch.from_numpy(a).cuda(), c_int, out=view)
        torch.cuda.synchronize()
        got = dst.cpu().numpy()
        assert int((got[shift:].reshape(rows, cols + 8)[:, :cols] != want).sum()) == 0, (rows, c_int)
        assert (got[:shift] == 7).all() and (got[shift:].reshape(rows, cols + 8)[:, cols:] == 7).all(), (rows, c_int)
    ia.close()
