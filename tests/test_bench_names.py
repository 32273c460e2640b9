"""What bench.py says about the kernel it has timed."""
import pytest

import bench
from paper_2601_21198_amd import synth, zipmoe as zm


@pytest.mark.parametrize("count,max_len,name", [
    (3, 8, "zm_decode_few_kernel<false, 2, kStreaming, kFitting>"), (6, 8, "zm_decode_few_kernel<false, 2, kStreaming, kFitting>"),
    (12, 8, "zm_decode_kernel<false, 2, kStreaming, kMany>"), (3, 12, "zm_decode_few_kernel<true, 2, kStreaming, kFitting>"),
    (12, 12, "zm_decode_kernel<true, 2, kStreaming, kMany>")])
def test_kernel_names(count, max_len, name):
    info = zm.blob_info(zm.compress(synth.special_tensor("gauss" if max_len == 8 else "wide", 50000, 3), 16384, 4096, max_len)[0])
    n = 1408 * 2048
    info.n_values, info.n_chunks = n, -(-n // info.chunk_values)
    info.sm_offset = (info.table_offset + info.table_stride * (info.n_chunks + 1) + 255) // 256 * 256
    info.e_offset = info.sm_offset + (n + 255) // 256 * 256
    info.blob_size = info.e_offset + n // 3 // 256 * 256
    assert bench.kernel_names([info] * count, zm.decode_launch_shapes([info] * count, zm.STORES_STREAMING)) == [name]


@pytest.mark.parametrize("stream_values,rows,says", [(512, 96, ""), (512, 1408, ", 8 streams a wave"), (1024, 1280, ", 4 streams a wave"), (1024, 1408, ""),
                                                     (2048, 1408, ", 2 streams a wave"), (2048, 4096, ""), (4096, 1408, "")])
def test_kernel_names_tell_waves_of_several_streams(stream_values, rows, says):
    info = zm.blob_info(zm.compress(synth.special_tensor("gauss", 50000, 3), 16384, stream_values, 8)[0])
    n = rows * 2048
    info.n_values, info.n_chunks = n, -(-n // info.chunk_values)
    info.sm_offset = (info.table_offset + info.table_stride * (info.n_chunks + 1) + 255) // 256 * 256
    info.e_offset = info.sm_offset + (n + 255) // 256 * 256
    info.blob_size = info.e_offset + n * 2 // 5 // 256 * 256
    name, = bench.kernel_names([info] * 6, zm.decode_launch_shapes([info] * 6, zm.STORES_STREAMING))
    assert name.startswith("zm_decode_few_kernel<false, 2, kStreaming") and name.partition(">")[2] == says


def test_traffic_is_reported_for_what_it_was_measured_with(monkeypatch):
    monkeypatch.setitem(bench.MEASURED_TRAFFIC, "kernel_sha256_16", bench.kernel_sha256_16())
    assert bench.measured_traffic("cfg4") == bench.MEASURED_TRAFFIC["bytes_per_launch"]["cfg4"]
    assert bench.measured_traffic("cfg4", max_len=12) is None and bench.measured_traffic("cfg4", stream_values=1024) is None
    monkeypatch.setitem(bench.MEASURED_TRAFFIC, "kernel_sha256_16", "0" * 16)
    assert bench.measured_traffic("cfg4") is None
