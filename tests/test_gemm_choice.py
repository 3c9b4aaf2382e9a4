"""Which tile and split of K the packed-weight GEMM takes, asked of the library's own rule on the host (csrc/gemm_choice.h, plain C++): the tile
tests on the GPU run the tiles that they name, and no shape is given to a kernel that refuses it."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2501_06589_amd", "csrc", "gemm_choice.h")
TILES = ["64x64", "64x128", "128x64", "128x128", "128x256", "256x256", "duo 128", "duo 192", "duo 256"]
STORE, SWIGLU, QKV, RESIDUAL = range(4)


class Rule:
    def __init__(self, lib):
        self.lib = lib
        lib.split.argtypes = [C.c_int] * 4 + [C.c_float]

    def tile(self, m, n, k, epilogue=STORE, peers=0, ks=1, ldx=None):
        return TILES[self.lib.tile(m, n, k, ldx or k, epilogue, peers, ks)]

    def few(self, m, n, k):
        """Tile and split of a projection of at most 1024 rows that leaves partial products."""
        ks = self.lib.split(m, n, k, min(8, 2048 // m), 0.0)
        return self.tile(m, n, k, ks=ks), ks

    def reaches(self, ldx, k, jt):
        return bool(self.lib.reaches(ldx, k, jt))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    at = tmp_path_factory.mktemp("choice")
    (at / "rule.cpp").write_text(f'''#include "{HEADER}"
extern "C" int tile(int M, int N, int K, int ldx, int epilogue, int peers, int ks) {{ return gemm_best_tile(GemmShape{{M, N, K, ldx, epilogue, peers}}, ks, nullptr); }}
extern "C" int split(int M, int N, int K, int most, float extra) {{ return gemm_best_split(M, N, K, most, extra); }}
extern "C" int reaches(int ldx, int K, int jt) {{ return gemm_duo_reaches(ldx, K, jt); }}
''')
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-o", str(at / "rule.so"), str(at / "rule.cpp")], check=True)
    return Rule(C.CDLL(str(at / "rule.so")))


def test_the_gpu_tests_run_the_tiles_that_they_name(rule):
    # test_gpu_few_rows.py
    assert rule.tile(257, 2 * 4160, 4160, SWIGLU) == "duo 128"
    assert rule.few(513, 2112, 8256) == ("duo 128", 3)
    assert rule.tile(700, 2 * 8256, 576, SWIGLU) == "duo 256"
    assert rule.tile(1025, 4160, 1088, RESIDUAL, 9) == "duo 192"
    assert rule.tile(2100, (16 + 2 * 2) * 128, 1088, QKV) == "duo 192"
    for n, k, epilogue in (((16 + 2 * 2) * 128, 2112, QKV), (2112, 2048, RESIDUAL), (2 * 2112, 2112, SWIGLU), (2112, 2112, RESIDUAL)):
        assert rule.tile(3000, n, k, epilogue, 2) == "duo 256"
    assert rule.tile(1101, 4128, 2080, RESIDUAL, 4) == "128x256"
    assert rule.tile(4100, 2112, 512, RESIDUAL) == "256x256"
    for rows in (385, 400, 500):
        assert rule.tile(rows, 2 * 14304, 2112, SWIGLU) == "256x256"
    # test_gpu_parity.py, 13200 rows
    assert [rule.tile(13200, *a) for a in ((768, 1056, QKV), (1056, 512, RESIDUAL, 3), (2048, 1056, SWIGLU), (1056, 1024, RESIDUAL, 3))] == [
        "128x128", "duo 128", "128x256", "duo 128"]
    assert [rule.tile(13200, *a) for a in ((768, 1024, QKV), (1024, 512, RESIDUAL, 3), (2368, 1024, SWIGLU), (1024, 1184, RESIDUAL, 3))] == [
        "256x256", "duo 256", "duo 192", "128x256"]
    for peers in (2, 7):
        assert rule.tile(13200, 1056, 512, RESIDUAL, peers) == rule.tile(13200, 1056, 1024, RESIDUAL, peers) == "duo 128"


def test_no_tile_takes_a_shape_that_its_kernel_refuses(rule):
    """Offsets of the 128-row tiles' requests are 32 bits: K or a row stride of 2^23 and more, K x columns beyond 2^31 bytes; 256 x 256 and
    those tiles want whole stages of 64 k, and no split or no few rows."""
    bits = 0x7fffffff
    for k in (64, 4096, 8256, 8_200_000, 8_323_136, 8_388_608, 8_500_032, 9_000_000, 16_777_216, 22_400_000):
        for jt in (2, 3, 4):
            assert rule.reaches(k, k, jt) == (128 * k * 2 + k * 2 <= bits and jt * (k // 32) * 1024 <= bits)
        for m in (257, 1024, 4001):
            for n in (32, 512, 4096):
                for epilogue, peers in ((STORE, 0), (SWIGLU, 0), (RESIDUAL, 0), (RESIDUAL, 7)):
                    t = rule.tile(m, n, k, epilogue, peers)
                    if t.startswith("duo"):
                        assert k % 64 == 0 and rule.reaches(k, k, int(t[4:]) // 64)
                    if t == "256x256":
                        assert k % 64 == 0 and k >= 256 and not (epilogue == RESIDUAL and peers)
                    assert not (t == "64x64" and epilogue == RESIDUAL)
    assert rule.tile(4001, 4096, 4096, RESIDUAL, 7).startswith("duo")
    assert not rule.tile(4001, 4096, 9_000_000 // 64 * 64, RESIDUAL, 7).startswith("duo")
    for m in (17, 256):
        assert not rule.tile(m, 4096, 4096).startswith("duo")
    for k in (32, 96, 2080):
        assert rule.tile(2048, 4096, k) in TILES[:5]
