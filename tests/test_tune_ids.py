"""Ids of tile configurations stand in saved tuning tables: each names the tile it always
has (no GPU needed)."""
import pytest

FIRST = {0: [(128, 16), (128, 32), (64, 64), (64, 128), (64, 128), (128, 64), (64, 64)],       # FP64
         16: [(128, 16), (128, 32), (64, 64), (128, 64), (64, 32)]}                            # batched FP64


@pytest.mark.parametrize("compute", FIRST)
def test_ids_keep_their_tiles(compute):
    from paper_2406_18001_amd import kdcd as K
    got = [c[:2] for c in K.kdcd_tune_configs(compute)]
    assert got[:len(FIRST[compute])] == FIRST[compute]
    assert (64, 16) in got and (64, 32) in got


def test_saved_table_of_the_first_ids(tmp_path):
    from paper_2406_18001_amd import kdcd as K
    path = tmp_path / "tune.txt"
    path.write_text("".join(f"{c} {900 + i} 512 {i}\n" for c in FIRST for i in range(len(FIRST[c]))))
    K.kdcd_tune_load(path)
    try:
        for c in FIRST:
            for i, tile in enumerate(FIRST[c]):
                assert K.kdcd_tune_configs(c)[K.kdcd_tune_get(c, 900 + i, 512)][:2] == tile
    finally:
        for c in FIRST:
            for i in range(len(FIRST[c])):
                K.kdcd_tune_set(c, 900 + i, 512, -1)
