"""Which tiles an LM head of 65 to 256 rows takes (csrc/long_plan.h), compiled for the host: at sizes over the range of vocabularies the
choice is near the fastest of the forms as they were measured, and the calls of test_gpu_lm_head_rows.py reach the tiles they are for."""
import ctypes
import subprocess

import pytest

from paper_2604_11554_amd import build

import test_gpu_lm_head_rows as G

SOURCE = """
#include "long_plan.h"
extern "C" int form(int V, int K, int T, int units) { return rlx::long_lmhead_form(V, K, T, units); }
extern "C" int part_tiles(int form) { return rlx::long_lmhead_part_tiles(form); }
extern "C" int forms(int i) { const int f[] = {rlx::LONG_512x128, rlx::LONG_128x128, rlx::LONG_320x128, rlx::LONG_320x256}; return f[i]; }
"""
# us of a decode step of two or three layers on 256 units (medians of 56, one draw per row, no logits): K, vocabulary, rows: 512 x 128,
# 128 x 128, 320 x 128, 320 x 256
MEASURED = {
    (2560, 16000, 65): (388, 327, 359, 374), (2560, 16000, 96): (427, 367, 394, 414), (2560, 16000, 128): (488, 429, 449, 468),
    (2560, 16000, 129): (539, 477, 500, 555), (2560, 16000, 192): (603, 540, 565, 627), (2560, 16000, 256): (656, 598, 620, 685),
    (2560, 32000, 65): (389, 333, 360, 376), (2560, 32000, 96): (428, 372, 396, 415), (2560, 32000, 128): (493, 439, 456, 474),
    (2560, 32000, 129): (545, 504, 505, 558), (2560, 32000, 192): (608, 571, 576, 628), (2560, 32000, 256): (666, 633, 634, 693),
    (2560, 100352, 65): (422, 453, 463, 496), (2560, 100352, 96): (468, 495, 507, 539), (2560, 100352, 128): (533, 557, 583, 602),
    (2560, 100352, 129): (683, 666, 666, 700), (2560, 100352, 192): (756, 746, 752, 793),
    (2560, 100352, 256): (820, 825, 821, 875), (2560, 128256, 65): (443, 458, 472, 503), (2560, 128256, 96): (488, 507, 517, 549),
    (2560, 128256, 128): (562, 576, 596, 611), (2560, 128256, 129): (715, 705, 749, 706),
    (2560, 128256, 192): (782, 783, 841, 809), (2560, 128256, 256): (845, 865, 907, 882),
    (2560, 151936, 65): (561, 517, 491, 523), (2560, 151936, 96): (597, 550, 524, 554), (2560, 151936, 128): (673, 614, 606, 621),
    (2560, 151936, 129): (824, 770, 758, 721), (2560, 151936, 192): (894, 850, 852, 816),
    (2560, 151936, 256): (948, 933, 917, 898), (2560, 200064, 65): (563, 572, 560, 610), (2560, 200064, 96): (612, 622, 603, 654),
    (2560, 200064, 128): (692, 691, 692, 720), (2560, 200064, 129): (954, 873, 839, 854),
    (2560, 200064, 192): (1026, 953, 945, 962), (2560, 200064, 256): (1089, 1051, 1017, 1049),
    (2048, 151936, 96): (844, 791, 777, 798), (2048, 151936, 112): (874, 808, 816, 816),
    (2048, 151936, 128): (870, 809, 816, 814), (2048, 151936, 129): (999, 938, 940, 902),
    (2048, 151936, 256): (1135, 1114, 1108, 1090), (2048, 24000, 90): (683, 637, 656, 673),
    (2048, 24000, 220): (854, 819, 822, 879), (2048, 140000, 90): (810, 778, 759, 777),
    (2048, 140000, 220): (1089, 1041, 1042, 1033), (4096, 32000, 80): (591, 515, 541, 570),
    (4096, 32000, 256): (890, 839, 841, 931), (4096, 128256, 80): (701, 716, 725, 764),
    (4096, 128256, 256): (1153, 1198, 1229, 1207), (4096, 151936, 80): (854, 778, 733, 778),
    (4096, 151936, 256): (1318, 1320, 1277, 1258), (1024, 100352, 96): (379, 389, 400, 421),
    (1024, 100352, 128): (448, 459, 472, 486), (1024, 100352, 256): (699, 694, 701, 730),
    (1024, 151936, 96): (456, 425, 416, 436), (1024, 151936, 128): (552, 496, 502, 506),
    (1024, 151936, 256): (778, 754, 761, 748), (3072, 81793, 100): (496, 494, 478, 475), (3072, 81793, 250): (838, 784, 767, 759),
    (3072, 110000, 100): (516, 532, 554, 573), (3072, 110000, 250): (849, 865, 852, 915),
}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("lm")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC, str(d / "plan.cpp"), "-o", str(d / "plan.so")],
                   check=True, capture_output=True)
    return ctypes.CDLL(str(d / "plan.so"))


@pytest.mark.parametrize("size", MEASURED)
def test_the_form_is_near_the_fastest(lib, size):
    K, V, T = size
    us = dict(zip(map(lib.forms, range(4)), MEASURED[size]))
    lm_head = max(2 * K * V / 6.6e6, 4 * K * V * T / 1.35e9)      # at the card's rates: its weights, or both terms' products
    # the vocabulary alone moves the fastest form: taking one by the rows alone was up to three times the LM head's time behind
    assert us[lib.form(V, K, T, 256)] <= min(us.values()) + 0.1 * lm_head, us


def test_the_compared_calls_reach_their_tiles(lib):
    wide = {lib.forms(2), lib.forms(3)}
    taken = {(T, lib.form(V, K, T, 256)) for T, V, K in G.WIDE_TILES}
    assert {f for _, f in taken} == wide, taken
    assert all(lib.form(V, K, T, 256) == lib.forms(1) for V, K in ((353, 80), (705, 48), (161, 272)) for T in (96, 200, 256))
    # more rows than that: the two forms without wide parts, whose 64 ids a part are what the partials' buffer is sized for
    for T in (257, 500, 1024):
        for V in (353, 32000, 151936):
            assert lib.part_tiles(lib.form(V, 2560, T, 256)) == 2
    assert [lib.part_tiles(lib.forms(i)) for i in range(4)] == [2, 2, 5, 5]
