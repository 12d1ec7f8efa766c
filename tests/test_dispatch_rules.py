"""The host's rules that pick a kernel by sizes, against measured times of both sides (MI355X, us per call): what
a rule takes is never slower than the side it leaves by more than two runs of one side differ."""
import ctypes as C

import pytest

import paper_2404_00509_amd as mae

NOISE = 1.05


def embed_tile(M, D, E):
    rule = mae.load()._ZN3mae10embed_tileElii
    rule.argtypes, rule.restype = (C.c_int64, C.c_int, C.c_int), C.c_int
    return rule(M, D, E)


# rows, D, E: patch embedding by tiles of 256 x 256 and of 128 x 128, and by the large tile as it was when
# it was the only one
@pytest.mark.parametrize("M,D,E,large,small,only", [
    (12544, 768, 768, 27.3, 27.4, 28.8), (15360, 768, 768, 27.4, 28.0, 29.1), (18432, 768, 768, 28.4, 33.0, 30.5),
    (20480, 768, 768, 29.7, 34.0, 31.8), (21760, 768, 768, 30.8, 35.1, 32.9), (22528, 768, 768, 52.7, 42.5, 55.5),
    (25600, 768, 768, 52.1, 43.8, 54.5), (32768, 768, 768, 52.5, 51.7, 56.3), (36608, 768, 768, 53.8, 58.8, 58.3),
    (39936, 768, 768, 56.4, 64.1, 60.8), (43520, 768, 768, 60.0, 67.3, 64.8), (56320, 768, 768, 83.8, 90.5, 91.5),
    (13824, 588, 1024, 25.9, 31.8, 28.9), (16384, 588, 1024, 28.2, 33.5, 30.6), (19200, 588, 1024, 46.8, 41.1, 51.8),
    (27392, 588, 1024, 48.6, 57.6, 54.1), (32512, 588, 1024, 53.4, 65.4, 60.2), (9216, 1200, 1024, 36.7, 43.2, 42.2),
    (13824, 1200, 1024, 40.2, 51.5, 44.3), (16384, 1200, 1024, 44.0, 56.4, 46.9), (19200, 1200, 1024, 75.5, 71.1, 81.2),
    (29952, 1200, 1024, 81.8, 104.7, 88.8), (13824, 768, 1000, 28.7, 33.3, 30.2), (27392, 768, 1000, 54.1, 60.1, 57.4),
    (30720, 192, 384, 15.0, 13.0, 15.8), (55040, 192, 384, 26.9, 21.9, 29.4), (11008, 3072, 1280, 83.8, 102.4, 83.1),
    (2048, 768, 768, 24.4, 10.2, 25.7), (5120, 768, 768, 25.7, 11.6, 26.9), (87296, 768, 768, 119.4, 137.3, 126.2)])
def test_tiles_of_the_embedding(M, D, E, large, small, only):
    side = embed_tile(M, D, E)
    if side == 64:  # not more than 128 blocks of 128 x 128: faster than either of both
        assert -(-M // 128) * -(-E // 128) < 128
        return
    taken = {256: large, 128: small}[side]
    assert taken <= NOISE * min(large, small)
    assert taken <= 1.01 * only


def test_tiles_of_the_embedding_at_the_ends_of_its_range():
    assert embed_tile(1, 4, 1) == 64
    assert embed_tile(1 << 28, 3072, 8192) == 256
    assert embed_tile(1 << 28, 4, 1) == 256
    for D in (4, 64, 588, 3072):  # beyond two rounds
        assert embed_tile(256 * 513, D, 256) == 256


OUTPUTS, LOSS, AUGMENT = 0, 1, 2
ALL_ROWS = 0x7FFFFFFF


def staged_rows(B, S, p, side, use):
    rule = mae.load()._ZN3mae15crop_whole_rowsEiiiiNS_7CropUseE
    rule.argtypes, rule.restype = (C.c_int,) * 5, C.c_int
    return rule(B, S, p, side, use)


# images, their side, output, patch: all rows between the first and the last that is tapped, or pairs of rows
@pytest.mark.parametrize("use,B,side,S,p,whole,pairs", [
    (OUTPUTS, 512, 500, 224, 16, 87.9, 89.2), (OUTPUTS, 64, 500, 224, 16, 20.0, 20.7),
    (OUTPUTS, 512, 500, 240, 16, 94.0, 95.6), (OUTPUTS, 1024, 256, 112, 16, 43.9, 44.7),
    (OUTPUTS, 512, 500, 224, 14, 91.7, 83.1), (OUTPUTS, 64, 500, 224, 14, 20.5, 20.9),
    (OUTPUTS, 1024, 256, 112, 14, 46.2, 42.8), (OUTPUTS, 64, 256, 112, 14, 12.8, 13.2),
    (OUTPUTS, 1024, 256, 112, 8, 63.8, 59.1), (OUTPUTS, 64, 256, 112, 8, 15.7, 15.4),
    (OUTPUTS, 512, 500, 192, 16, 134.0, 122.4), (OUTPUTS, 64, 500, 192, 16, 25.3, 23.6),
    (OUTPUTS, 512, 500, 192, 12, 170.5, 126.8), (OUTPUTS, 64, 500, 192, 12, 27.4, 25.6),
    (OUTPUTS, 512, 500, 160, 16, 150.8, 101.5), (OUTPUTS, 512, 500, 128, 8, 191.8, 140.6),
    (OUTPUTS, 1024, 256, 64, 4, 53.6, 39.5), (OUTPUTS, 512, 500, 224, 28, 215.0, 247.0),
    (OUTPUTS, 512, 500, 192, 24, 144.3, 170.4), (OUTPUTS, 512, 500, 224, 32, 188.9, 203.5),
    (OUTPUTS, 512, 500, 200, 20, 152.1, 174.1), (OUTPUTS, 1024, 256, 120, 20, 94.9, 108.0),
    (LOSS, 512, 500, 224, 16, 224.7, 227.5), (LOSS, 64, 500, 224, 16, 47.2, 48.1),
    (LOSS, 512, 500, 192, 16, 273.3, 198.7), (LOSS, 512, 500, 224, 14, 244.8, 239.8),
    (AUGMENT, 512, 500, 224, 16, 254.3, 256.5), (AUGMENT, 64, 500, 224, 16, 43.6, 44.4),
    (AUGMENT, 512, 500, 224, 14, 308.1, 283.2), (AUGMENT, 512, 500, 240, 16, 280.1, 283.2),
    (AUGMENT, 512, 500, 224, 32, 388.8, 324.9), (AUGMENT, 512, 500, 200, 20, 286.7, 254.9),
    (AUGMENT, 1024, 256, 120, 20, 219.3, 223.3), (AUGMENT, 512, 500, 224, 28, 463.3, 443.9)])
def test_staged_rows_of_large_crops(use, B, side, S, p, whole, pairs):
    rows = staged_rows(B, S, p, side, use)
    assert rows in (2 * p, ALL_ROWS)
    assert (whole if rows == ALL_ROWS else pairs) <= 1.001 * min(whole, pairs)


def test_staged_rows_of_the_loss_and_the_augmentation_do_not_depend_on_the_batch():
    # (partial sums are kept per column part, of which a shard has as many as the whole batch)
    for use in (LOSS, AUGMENT):
        for S, p in ((112, 14), (224, 14), (224, 16), (224, 32), (120, 20), (112, 8)):
            for side in (256, 500):
                assert len({staged_rows(B, S, p, side, use) for B in (1, 64, 512, 4096)}) == 1
