"""Which kernel a launch takes (zipmoe_kinds.h, built as host code): at the lines between the kinds, and for what a line could miss."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "zipmoe_kinds.h"
// long_codes streaming {stream_values n_streams last_values e_size}...
int main(int argc, char **argv)
{
    static const char *const names[] = {"short", "sparse", "fitting", "many", "mixed", "deep"};
    zipmoe::Streams s;
    for (int i = 3; i + 3 < argc; i += 4)
        s.add(std::strtoul(argv[i], nullptr, 10), std::strtoul(argv[i + 1], nullptr, 10), std::strtoul(argv[i + 2], nullptr, 10), std::strtoull(argv[i + 3], nullptr, 10));
    const bool long_codes = argv[1][0] == '1';
    const zipmoe::Stores stores = argv[2][0] == '1' ? zipmoe::kStreaming : zipmoe::kThrough;
    const zipmoe::Kind k = zipmoe::kind_of(long_codes, s, stores);
    std::printf("%s %d %d\n", names[k], zipmoe::most_waves(k, long_codes), zipmoe::pairs_ahead(k, long_codes, stores));
}
"""


@pytest.fixture(scope="module")
def kind_of(tmp_path_factory):
    at = tmp_path_factory.mktemp("kinds")
    (at / "kinds.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2601_21198_amd", "csrc"), str(at / "kinds.cpp"), "-o", str(at / "kinds")])

    def ask(tensors, long_codes=False, streaming=False, bits=3):
        """tensors: (stream_values, streams), whole streams of `bits` bits of code a value; bits = 8: stored raw"""
        args = [str(x) for w, n in tensors for x in (w, n, w, w * n * bits // 8 + (256 if bits == 8 else 0))]
        name, waves, ahead = subprocess.check_output([str(at / "kinds"), str(int(long_codes)), str(int(streaming)), *args], text=True).split()
        return name, int(waves), int(ahead)
    return ask


@pytest.mark.parametrize("streaming", [False, True])
@pytest.mark.parametrize("w", [4608, 5632, 6144, 7680])
@pytest.mark.parametrize("n", [100, 2000, 20000])
def test_streams_of_no_whole_groups_keep_their_waves(kind_of, w, n, streaming):
    """they never decode straight through, so that the three waves of long streams starve them"""
    assert kind_of([(w, n)], streaming=streaming)[:2] == ("fitting", 7)
    assert kind_of([(w, n)], long_codes=True, streaming=streaming)[1] >= 5
    assert kind_of([(8192, n)], streaming=streaming) == ("deep", 3, 4)


@pytest.mark.parametrize("streaming", [False, True])
def test_raw_launches_keep_their_waves(kind_of, streaming):
    assert kind_of([(4096, 12288)], streaming=streaming)[:2] == ("many", 3)
    assert kind_of([(4096, 12288)], streaming=streaming, bits=7)[:2] == ("many", 3)       # dense codes are no raw chunks
    assert kind_of([(4096, 12288)], streaming=streaming, bits=8)[:2] == ("fitting", 7)


def test_long_codes_find_places_or_are_served_straight_through(kind_of):
    assert kind_of([(4096, 4608)], long_codes=True, streaming=True) == ("fitting", 5, 4)
    assert kind_of([(4096, 4608)], long_codes=True) == ("fitting", 5, 1)
    assert kind_of([(4096, 7168)], long_codes=True, streaming=True) == ("fitting", 5, 4)
    assert kind_of([(4096, 7169)], long_codes=True, streaming=True) == ("many", 4, 4)
    assert kind_of([(4096, 5120)], long_codes=True) == ("fitting", 5, 1)
    assert kind_of([(4096, 5121)], long_codes=True) == ("many", 4, 1)
    for w in (1536, 2048, 3584):
        assert kind_of([(w, 8192)], long_codes=True) == ("short", 8, 2)
        assert kind_of([(w, 8193)], long_codes=True)[:2] == ("fitting", 5)
    assert kind_of([(1024, 50000)], long_codes=True) == ("short", 8, 2)


@pytest.mark.parametrize("streaming", [False, True])
def test_launches_of_several_stream_lengths(kind_of, streaming):
    # whole groups of one and of several
    assert kind_of([(8192, 256)] + [(4096, 512)] * 23, streaming=streaming) == ("mixed", 6, 4 if streaming else 2)
    assert kind_of([(8192, 256)] + [(1024, 2048)] * 23, streaming=streaming)[0] == "mixed"
    assert kind_of([(8192, 256)] * 8 + [(4096, 512)] * 4, streaming=streaming)[0] == ("deep" if streaming else "mixed")
    assert kind_of([(8192, 256)] * 7 + [(4096, 512)] * 4, streaming=streaming)[0] == "mixed"
    assert kind_of([(8192, 256), (16384, 128)], streaming=streaming)[0] == "deep"
    # one group and shorter ones: the more frequent decide
    assert kind_of([(4096, 512)] * 23 + [(1024, 2048)], streaming=streaming)[0] == "mixed"
    assert kind_of([(4096, 512)] + [(1024, 2048)] * 23, streaming=streaming)[:2] == ("fitting", 7)
    assert kind_of([(6144, 342)] * 8 + [(4096, 512)] * 5, streaming=streaming)[0] == "fitting"
    assert kind_of([(10240, 20000)], streaming=streaming)[0] == "mixed"
    # long codes have no kind of their own for these
    assert kind_of([(8192, 256)] + [(4096, 512)] * 23, long_codes=True, streaming=streaming)[0] == "deep"
    assert kind_of([(4096, 512)] * 23 + [(1024, 2048)], long_codes=True, streaming=streaming)[0] == "fitting"


def test_few_streams_ask_early_more_ask_late(kind_of):
    assert kind_of([(4096, 1024)] * 3) == ("sparse", 7, 2)
    assert kind_of([(4096, 3073)]) == ("fitting", 7, 1)
    assert kind_of([(4096, 3072)], streaming=True) == ("fitting", 7, 2) == kind_of([(4096, 3073)], streaming=True)
    assert kind_of([(4096, 1024)], long_codes=True) == ("sparse", 5, 4)
    assert kind_of([(4096, 1025)], long_codes=True) == ("fitting", 5, 1)
    assert kind_of([(4096, 7169)]) == ("many", 3, 2)


@pytest.mark.parametrize("streaming", [False, True])
def test_nearly_whole_groups_run_seven_waves(kind_of, streaming):
    assert kind_of([(2048, 30000)], streaming=streaming) == ("short", 8, 2)
    for w in (2560, 3584):
        assert kind_of([(w, 20000)], streaming=streaming)[:2] == ("fitting", 7)
