"""What a cache fetch moves and from where, on zipmoe_cache.hip built as host code with a model of the runtime that knows
which host memory a kernel could reach (tests/cache_on_host)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = os.environ.get("HOST_CLANG", "/opt/rocm/llvm/bin/clang++")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    here = os.path.join(ROOT, "tests", "cache_on_host")
    exe = str(tmp_path_factory.mktemp("cache") / "cache_on_host")
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-x", "c++", "-I", here, "-I", os.path.join(ROOT, "paper_2601_21198_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), os.path.join(here, "cache_on_host.cpp"), "-o", exe])
    return exe


def fetch(program, *scenario):
    """(bytes that differ, parts by kernel, parts by copy, reads of unmapped memory, misaligned parts)"""
    return tuple(int(x) for x in subprocess.check_output([program, *scenario], text=True).split())


@pytest.mark.parametrize("source,parts", [("blobs", 4), ("packed", 2)])
def test_mapped_memory_is_read_by_the_kernel_and_pageable_memory_is_copied(program, source, parts):
    assert fetch(program, "whole", source) == (0, parts, 0, 0, 0)
    assert fetch(program, "pageable", source) == (0, 0, parts, 0, 0)


def test_parts_that_are_no_whole_vectors_are_copied_to_their_last_byte(program):
    """descriptions of blobs laid out by hand: an E region that ends off a multiple of 16, sections that start off one"""
    assert fetch(program, "odd-end", "blobs") == (0, 2, 2, 0, 0)
    assert fetch(program, "odd-sections", "blobs") == (0, 0, 4, 0, 0)
    # an image's regions are whole vectors whatever the blobs are
    assert fetch(program, "odd-end", "packed") == (0, 2, 0, 0, 0)
    assert fetch(program, "odd-sections", "packed") == (0, 2, 0, 0, 0)


@pytest.mark.parametrize("source,parts", [("blobs", 4), ("packed", 2)])
def test_the_kernel_reads_nothing_that_is_not_mapped_when_the_fetch_is_issued(program, source, parts):
    # unpinned after the cache was made, and still valid
    assert fetch(program, "unmapped-later", source) == (0, 0, parts, 0, 0)
    # first and last page mapped, by an allocation each, and pageable memory between them: what lies in the last page alone
    # is the blobs' E regions
    assert fetch(program, "hole", source) == ((0, 2, 2, 0, 0) if source == "blobs" else (0, 0, 2, 0, 0))


@pytest.mark.parametrize("source", ["blobs", "packed"])
@pytest.mark.parametrize("memory", ["whole", "pageable"])
@pytest.mark.parametrize("ends", ["decoded", "refused", "captured"])
def test_what_a_fetch_has_issued_is_over_when_the_cache_is_gone(program, source, memory, ends):
    """a fetch that is decoded, one whose decode is refused behind the fetch, and one issued before another is captured: (something was
    under way, copies and launches that destruction has not waited for, bytes that differ)"""
    assert fetch(program, memory, source, ends) == (1, 0, 0)
