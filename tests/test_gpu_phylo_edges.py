"""Trees at the edges of the reconstruction's tiles: chunks of 2,048 sorted
entries merged by rank, tiles of 1,024 boundaries and the table levels above
them -- one entry more and fewer, many equal keys across chunks, and an
annotation of all ones, whose key equals the padding's.  Canonical Newick
text, character for character, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 1024, 1025, 2047, 2048, 2049, 2050, 3073, 4096, 4097, 8193])
@pytest.mark.parametrize("values", ["spread", "few"])
def test_tree_at_tile_edges(orc, n, values):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_10861_amd as hs
    rng = np.random.default_rng(n)
    T = 5000
    words = rng.integers(0, 2**32, size=(n, 2), dtype=np.uint64).astype(np.uint32)
    if values == "few":
        words = words[rng.integers(0, min(n, 7), size=n)]
        words[-1] = 0xffffffff
    cnt = np.full(n, T, np.uint32)
    tree = hs.phylo_tree("hybrid", 64, torch.from_numpy(cnt.view(np.int32)).cuda(),
                         torch.from_numpy(words.view(np.int32)).cuda())
    assert tree["status"] == 0
    assert hs.newick(tree) == orc.phylo_newick(2, 64, cnt, words)
