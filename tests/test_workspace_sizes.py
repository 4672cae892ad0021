"""Workspaces of a size that served earlier still serve: the sizes that tsne_workspace_bytes and
tsne_workspace_bytes_implicit gave for 10 dimensions when a problem's force pass ran in whole tiles
and its search in groups of four row blocks."""
import os

import pytest

from paper_1812_09869_amd import _lib


@pytest.mark.parametrize("n,fp64,x3", [
    (2, (599808, 599808), (667392, 667392)),
    (256, (602368, 602368), (669952, 669952)),
    (257, (1996032, 1996032), (2131200, 2131200)),
    (1024, (7167232, 7167232), (7437568, 7437568)),
    (1025, (9643264, 9643264), (9981184, 9981184)),
    (2048, (18658048, 18658048), (19198720, 19198720)),
    (2049, (22228224, 22228224), (22836480, 22836480)),
    (4096, (54618880, 54618880), (55700224, 55700224)),
    (4097, (60377088, 60377088), (61526016, 61526016)),
    (65536, (9180467712, 1093849600), (9197769216, 1111151104))])
def test_sizes_have_not_grown(n, fp64, x3):
    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("libtsne355.so not built")
    for mode, sizes in (("fp64", fp64), ("bf16x3", x3)):
        assert 0 < _lib.workspace_bytes(n, 10, mode) <= sizes[0]
        assert 0 < _lib.workspace_bytes_implicit(n, 10, mode) <= sizes[1]
