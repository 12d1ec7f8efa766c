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
