"""GPU parity of the many-row kernel where its blocks change: one row more than a block of 128 or 256, several blocks, rows
that leave most of the last block empty, and sequences of one tile, one key more, and many tiles over several splits (the
running reference of a row moves between tiles, is different in every split, and may lie far above a tile's scores).  Bar
and oracle as in test_gpu_parity.py."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_paged import run_paged_decode_case, run_paged_hybrid_case  # noqa: E402
from test_gpu_parity import run_decode_case  # noqa: E402


@pytest.mark.parametrize("d,bits", [(64, 4), (64, 1.5), (128, 3), (128, 4)])
@pytest.mark.parametrize("n_q,lens", [(128, [64]), (129, [65, 1]), (192, [1000]), (257, [640, 0, 63])])
def test_decode_many_rows_blocks(d, bits, n_q, lens):
    run_decode_case(d, bits, len(lens), 1, 1, n_q, lens, "bf16", seed=int(d + n_q), want_scores=False)


def test_decode_many_rows_several_splits():
    run_decode_case(128, 3, 1, 2, 2, 140, [5000], "bf16", seed=11, want_scores=False)


# d = 128 takes blocks of 256 rows only where they leave fewer tiles to walk in a row: 288 workgroups of 128 rows against 144
# of 256 (the last of which has 129 rows); 16 splits against 25
@pytest.mark.parametrize("n_seq,n_kv,n_q,lens", [(9, 8, 385, [130, 64, 65, 0, 1, 129, 128, 2, 63]), (1, 8, 130, [25600])])
def test_decode_many_rows_blocks_of_256_at_128(n_seq, n_kv, n_q, lens):
    run_decode_case(128, 3, n_seq, n_kv, n_kv, n_q, lens, "bf16", seed=n_q, want_scores=False)


# ... at every bit width (a wavefront stages 16 coordinates of a key: triplets straddle two of them, and at the two-class
# widths the boundary between the classes falls inside one's share), over pages, and with a window merged in
WIDE_LENS = [130, 64, 65, 0, 1, 129, 128, 2, 63]


@pytest.mark.parametrize("bits", [1, 1.5, 2, 2.5, 4])
def test_decode_many_rows_blocks_of_256_at_128_every_width(bits):
    run_decode_case(128, bits, 9, 8, 8, 385, WIDE_LENS, "bf16", seed=int(500 + 10 * bits), want_scores=False)


@pytest.mark.parametrize("bits", [1, 2.5, 3, 4])
def test_decode_many_rows_blocks_of_256_at_128_paged(bits):
    run_paged_decode_case(128, bits, 9, 8, 8, 385, WIDE_LENS, seed=int(600 + 10 * bits))


def test_decode_many_rows_blocks_of_256_at_128_paged_with_window():
    run_paged_hybrid_case(128, 3, 9, 8, 8, 385, WIDE_LENS, [32, 5, 0, 7, 32, 1, 16, 31, 2], 32, "bf16", seed=700)


# d = 64 with blocks of 512 rows (two blocks of 32 rows per wavefront): three of them, the last with 76 rows (wavefronts with one
# block and with none), at every width, over pages and with a window; and several splits with a last block of 288 rows, where a row's
# reference moves between tiles
@pytest.mark.parametrize("bits", [1, 1.5, 2, 2.5, 3, 4])
def test_decode_many_rows_blocks_of_512(bits):
    run_decode_case(64, bits, 9, 8, 8, 1100, WIDE_LENS, "bf16", seed=int(800 + 10 * bits), want_scores=False)


def test_decode_many_rows_blocks_of_512_several_splits():
    run_decode_case(64, 3, 1, 24, 24, 800, [3000], "bf16", seed=901, want_scores=False)


def test_decode_many_rows_blocks_of_512_paged_with_window():
    run_paged_hybrid_case(64, 4, 9, 8, 8, 1100, WIDE_LENS, [32, 5, 0, 7, 32, 1, 16, 31, 2], 32, "bf16", seed=902)
