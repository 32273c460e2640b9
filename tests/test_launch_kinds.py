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


BUNDLES = r"""
#include <cstdio>
#include <cstdlib>
#include "zipmoe_kinds.h"
// long_codes streaming {stream_values n_streams last_values e_size}...: streams that a wave takes, the kind of kernel, waves of every tensor
int main(int argc, char **argv)
{
    zipmoe::Streams s;
    for (int i = 3; i + 3 < argc; i += 4)
        s.add(std::strtoul(argv[i], nullptr, 10), std::strtoul(argv[i + 1], nullptr, 10), std::strtoul(argv[i + 2], nullptr, 10), std::strtoull(argv[i + 3], nullptr, 10));
    const zipmoe::Bundle b = zipmoe::bundle_of(argv[1][0] == '1', s, argv[2][0] == '1' ? zipmoe::kStreaming : zipmoe::kThrough);
    std::printf("%u %s", b.streams, b.streams == 1 ? "-" : b.kind == zipmoe::kMany ? "many" : b.kind == zipmoe::kFitting ? "fitting" : "?");
    for (int i = 3; i + 3 < argc; i += 4) std::printf(" %u", zipmoe::waves_of(std::strtoul(argv[i + 1], nullptr, 10), std::strtoul(argv[i + 2], nullptr, 10), b.streams));
    std::printf("\n");
}
"""


@pytest.fixture(scope="module")
def bundle_of(tmp_path_factory):
    at = tmp_path_factory.mktemp("bundles")
    (at / "bundles.cpp").write_text(BUNDLES)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2601_21198_amd", "csrc"), str(at / "bundles.cpp"), "-o", str(at / "bundles")])

    def ask(tensors, long_codes=False, streaming=False, e=None):
        """tensors: (stream_values, streams[, last_values]) with e bytes a stream in the E region: (streams a wave takes, kind, waves of every tensor)"""
        args = [str(x) for w, n, *last in tensors for x in (w, n, last[0] if last else w, n * (e if e is not None else 64 + w * 3 // 8))]
        streams, kind, *waves = subprocess.check_output([str(at / "bundles"), str(int(long_codes)), str(int(streaming)), *args], text=True).split()
        return int(streams), kind, [int(x) for x in waves]
    return ask


@pytest.mark.parametrize("long_codes,streaming,w,line,bundle,kind", [
    (False, False, 512, 9, 8, "fitting"), (False, True, 512, 9, 8, "fitting"), (True, False, 512, 9, 8, "many"), (True, True, 512, 9, 8, "many"),
    (False, False, 1024, 10, 4, "fitting"), (False, True, 1024, 8, 4, "fitting"), (True, False, 1024, 7, 4, "fitting"), (True, True, 1024, 7, 4, "fitting"),
    (False, False, 2048, 6, 2, "fitting"), (False, True, 2048, 5, 2, "fitting"), (True, False, 2048, 6, 2, "fitting"), (True, True, 2048, 4, 2, "fitting")])
def test_from_which_line_on_a_wave_takes_several_streams(bundle_of, long_codes, streaming, w, line, bundle, kind):
    ask = lambda tensors: bundle_of(tensors, long_codes, streaming)
    n = line * 1024
    assert ask([(w, n)])[:2] == (1, "-")
    assert ask([(w, n + 1)])[:2] == (bundle, kind)
    # the launch counts, not the tensor
    assert ask([(w, n // 4)] * 4)[:2] == (1, "-")
    assert ask([(w, n // 4)] * 3 + [(w, n // 4 + 1)])[:2] == (bundle, kind)


def test_large_launches_of_short_streams(bundle_of):
    for long_codes in (False, True):
        for streaming in (False, True):
            ask = lambda w, n: bundle_of([(w, n)], long_codes, streaming)[:2]
            assert ask(512, 1 << 20) == (8, "many" if long_codes else "fitting")
            assert ask(1024, 16 * 1024) == (4, "fitting")
            assert ask(1024, 16 * 1024 + 1) == ((4, "many") if long_codes else (1, "-"))
            assert ask(2048, 9 * 1024) == (2, "fitting")
            assert ask(2048, 9 * 1024 + 1) == ((2, "many") if long_codes else (1, "-"))


def test_launches_that_no_bundle_is_made_of(bundle_of):
    many = 1 << 15
    for w in (1536, 2560, 4096, 8192):
        assert bundle_of([(w, many)])[0] == 1
    assert bundle_of([(512, many), (1024, many)])[0] == 1                       # streams of two lengths
    assert bundle_of([(2048, 8192)], e=1024)[0] == 2 and bundle_of([(2048, 8192)], e=1025)[0] == 1
    assert bundle_of([(512, many)], e=79)[0] == 1 and bundle_of([(512, many)], e=80)[0] == 8
    # raw tensors: as many bytes in the E region as values
    assert bundle_of([(512, many)], e=511)[0] == 8 and bundle_of([(512, many)], e=512)[0] == 1


@pytest.mark.parametrize("w,bytes_,line,dense", [(512, 320, 9, 12), (1024, 464, 7, 12), (2048, 864, 6, 9)])
def test_launches_of_dense_long_codes_need_more_streams(bundle_of, w, bytes_, line, dense):
    """with stores that may stay cached; of 512 values whatever the stores"""
    for streaming in (False, True):
        late = dense if not streaming or w == 512 else line
        for e, at in ((bytes_, line), (bytes_ + 1, late)):
            if streaming and w == 2048:
                at = 4
            assert bundle_of([(w, at * 1024)], True, streaming, e)[0] == 1
            assert bundle_of([(w, at * 1024 + 1)], True, streaming, e)[0] == 4096 // w
    assert bundle_of([(w, {512: 10, 1024: 11, 2048: 8}[w] * 1024)], False, False, bytes_ + 1)[0] == 4096 // w        # four short codes always fit a window
    assert bundle_of([(1024, 1 << 15)], True, False, 577)[0] == 1 and bundle_of([(1024, 1 << 15)], True, True, 577)[0] == 4


@pytest.mark.parametrize("w,bundle", [(512, 8), (1024, 4), (2048, 2)])
def test_waves_of_tensors_that_are_no_whole_bundles(bundle_of, w, bundle):
    """every stream is in one bundle or has a wave of its own, and a cut-off one has"""
    tensors = [(w, 1 << 15)]
    for n in list(range(1, 2 * bundle + 2)) + [1000 * bundle - 1, 1000 * bundle, 1000 * bundle + 1]:
        tensors += [(w, n), (w, n, 1), (w, n, w - 8)]
    streams, _, waves = bundle_of(tensors, long_codes=True)
    assert streams == bundle
    for (_, n, *last), got in zip(tensors, waves):
        whole = n - (1 if last else 0)
        assert got == whole // bundle + whole % bundle + (1 if last else 0), (n, last)
