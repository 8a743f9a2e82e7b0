"""A descriptor whose workspace is sized for a batch serves calls with fewer items: what the call with more items needs covers the one with
fewer, although fewer heads get more partial states each."""
import pytest

from paper_2510_08318_amd import binding as L

NO_WGRADS, WGRADS = L.linattn_workspace_bytes, L.linattn_workspace_bytes_wgrads


@pytest.mark.parametrize("size_of,H,d,n,B", [(NO_WGRADS, 87, 64, 4742, 3), (NO_WGRADS, 121, 64, 7859, 3), (NO_WGRADS, 116, 128, 15714, 3),
                                             (NO_WGRADS, 40, 128, 75600, 2), (WGRADS, 87, 64, 4742, 3), (WGRADS, 93, 64, 2130, 3),
                                             (WGRADS, 76, 64, 6760, 4), (WGRADS, 12, 128, 4133, 4)])
def test_a_batch_covers_a_smaller_one(size_of, H, d, n, B):
    need = [size_of(b, H, n, d, L.PHI_HEDGEHOG, L.BF16) for b in (B - 1, B)]
    assert need[0] <= need[1], need
