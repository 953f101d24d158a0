"""How a decompression takes the outliers of a piece of 2048 elements in: a mailbox of one word per octet, a picture of
the piece where two share an octet or a tile has more than 64, a search in the stream of a long tile, stores over the
last, incomplete piece.  Values above 1 are planted where each way ends and the next begins; everything is compared
with the oracle bit for bit, as binary32 and in the tensor's own format."""
import numpy as np
import pytest
import torch

from helpers import bits_of, run_parity

pytestmark = pytest.mark.gpu

PLANTS = {
    "one_octet_full": lambda n: np.arange(8, 16),
    "two_in_an_octet_at_both_ends_of_a_piece": lambda n: np.array([0, 7, 2040, 2047, 2048, 2050, 4088, 4095]),
    "sixty_four_octets": lambda n: 8 * np.arange(64) + 3,
    "sixty_five_octets": lambda n: 8 * np.arange(65) + 5,
    "a_whole_piece": lambda n: np.arange(2048, 4096),
    "everything": lambda n: np.arange(n),
    "one_end_of_a_long_tile": lambda n: np.concatenate([np.arange(0, 300, 3), np.arange(n - 30, n)]),
    "every_29th": lambda n: np.arange(0, n, 29),
}
# (quantisation group, elements): tiles of 2048 and 4096 elements, tiles that are no multiples of a piece, an odd end
SHAPES = [(64, 3 * 2048 + 1000), (512, 4 * 2048), (4096, 3 * 4096 + 77), (8, 2048 * 2 + 9), (24, 4080 * 2 + 13), (344, 11008 + 5),
          (11008, 2 * 11008 + 2040), (16384, 2 * 16384 + 1)]


@pytest.mark.parametrize("gq,n", SHAPES)
@pytest.mark.parametrize("plant", sorted(PLANTS))
def test_outliers_of_a_piece(gq, n, plant):
    for bits, asym, dtype in ((4, 0, torch.bfloat16), (8, 1, torch.float16), (8, 0, torch.bfloat16)):
        g = torch.Generator().manual_seed(gq + n + bits)
        x = torch.rand(n, generator=g) - 0.5
        at = torch.from_numpy(PLANTS[plant](n))
        at = at[at < n]
        x[at] = (torch.rand(at.numel(), generator=g) + 2.0) * torch.sign(x[at] + 1e-9)
        x = x.to(dtype)
        print(f"[restore] {plant} gq={gq} n={n} bits={bits} asym={asym}", flush=True)
        oc, *_ = run_parity(x, dict(bits=bits, quant_group=gq, asym=asym, outlier_mode="abs", stat_group=0, thresh=1.0, topk=0))
        assert oc.n_out == at.numel()


def test_the_stream_of_a_piece_is_found_by_search():
    """STD over rows of 16384 values whose outliers crowd in one piece of eight."""
    rng = np.random.default_rng(5)
    x = torch.from_numpy(rng.standard_normal(3 * 16384).astype(np.float32))
    for first in (0, 5 * 2048 + 11, 16384 - 200):
        x[16384 + first:16384 + first + 190] = 9.0
    x[40:44] = 30.0
    x = x.to(torch.bfloat16)
    oc, *_ = run_parity(x, dict(bits=8, quant_group=128, asym=0, outlier_mode="std", stat_group=16384, thresh=4.0, topk=0))
    assert oc.n_out > 500 and bits_of(x).size == 3 * 16384
