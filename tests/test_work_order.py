"""How launches are split and ordered, on the host (CPU only): every (query head,
query block) of an attention launch once, longest rows first, and each XCD on few
KV heads; a selection launch of few long rows over enough waves."""

from __future__ import annotations

import ctypes
import subprocess

import numpy as np
import pytest

from paper_2609_20971_amd import build

SOURCE = r"""
#include "rbs_launch.hpp"
using namespace rbs;
extern "C" int choose(int n, int hq, int hkv, int row_bytes, int b, int M, int selected) {
  return work_order(n, hq, hkv, row_bytes, b, M, selected != 0);
}
extern "C" int line(int n, int hq, int hkv, int b, int M, int resident, int selected) {
  return queue_line(n, hq, hkv, b, M, resident, selected != 0);
}
extern "C" int choose_batch(int n, int hq, int hkv, int b, int blocks) { return batch_order(n, hq, hkv, b, blocks); }
extern "C" int tokens_a_wave(int b, int blocks, int rows) { return row_tokens(b, blocks, rows); }
// Query head and query block of every work slot of one sequence.
extern "C" void items(int M, int hq, int hkv, int order, int* h, int* i) {
  for (int s = 0; s < M * hq; ++s) work_of(s, M * hq, M, hq, hq / hkv, order, h[s], i[s]);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "order.hip").write_text(SOURCE)
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-host-only", "-I", build.CSRC, "-shared", str(d / "order.hip"),
                    "-o", str(d / "order.so")], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return ctypes.CDLL(str(d / "order.so"))


BY_GROUP, BY_ROW, BY_XCD_ROW = 0, 1, 2


def _items(lib, M, hq, hkv, order):
    h, i = np.full(M * hq, -1, np.int32), np.full(M * hq, -1, np.int32)
    lib.items(M, hq, hkv, order, h.ctypes.data_as(ctypes.c_void_p), i.ctypes.data_as(ctypes.c_void_p))
    return h, i


def _tiles(hkv):
    return 8 % hkv == 0 or hkv % 8 == 0


HEADS = [(1, 1), (2, 1), (7, 1), (8, 1), (12, 2), (16, 2), (28, 4), (32, 4), (8, 8), (40, 8), (64, 8), (16, 16),
         (32, 16), (3, 3), (6, 3), (20, 5), (36, 12)]


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("M", [1, 2, 5, 8, 31, 64, 513])
def test_every_item_once_and_longest_rows_first(lib, hq, hkv, M):
    for order in (BY_GROUP, BY_ROW) + ((BY_XCD_ROW,) if _tiles(hkv) else ()):
        h, i = _items(lib, M, hq, hkv, order)
        assert np.array_equal(np.unique(h.astype(np.int64) * M + i), np.arange(M * hq))
        if order != BY_GROUP:
            for x in range(8):  # in-order dispatch and each queue start an XCD's longest rows first
                assert (np.diff(i[x::8]) <= 0).all()


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("B", [64, 128])
@pytest.mark.parametrize("row_bytes", [512, 256])
def test_a_launch_of_many_items_keeps_an_xcd_to_few_kv_heads(lib, hq, hkv, B, row_bytes):
    """Past 3072 (FP8: 4096, or 8192) items an XCD (slots x, x + 8, ...) works on one KV
    head at a time, or on n_kv / 8 of its own, whatever the head counts."""
    for n in (8100, 16384, 40000, 65536, 131072):
        M = -(-n // B)
        order = lib.choose(n, hq, hkv, row_bytes, B, M, 0)
        assert order != BY_XCD_ROW or _tiles(hkv)
        if M * hq <= (3072 if row_bytes > 256 else 4096 if _tiles(hkv) else 8192):
            continue
        h, i = _items(lib, M, hq, hkv, order)
        for x in range(8):
            mine = (h // (hq // hkv))[x::8][i[x::8] >= 8]  # (the last, shortest rows may be anyone's)
            if order == BY_GROUP:  # one after another
                assert (np.diff(mine) >= 0).all()
            else:
                assert len(np.unique(mine)) <= max(1, hkv // 8), (n, x, np.unique(mine))


@pytest.mark.parametrize("hq,hkv", [(8, 8), (16, 16), (24, 8), (32, 32)])
@pytest.mark.parametrize("selected", [0, 1])
def test_kv_heads_that_fill_the_xcds_stay_on_them_at_64_token_blocks(lib, hq, hkv, selected):
    """From 1900 items of more than 96 blocks on, each XCD has KV heads of its own
    (up to 128 MiB of K and V, 256 with eight heads, 512 for selected lists) and
    the launch is queued."""
    for blocks in (97, 120, 240, 312, 750, 1024, 2048):
        n, items = 64 * blocks - 7, hq * blocks
        if items <= 1900 or n * hkv * 512 > (512 if selected else 256 if hkv == 8 else 128) << 20:
            continue
        assert lib.choose(n, hq, hkv, 512, 64, blocks, selected) == BY_XCD_ROW
        assert lib.line(n, hq, hkv, 64, blocks, 1024, selected) == 1900


@pytest.mark.parametrize("hq,hkv,tokens,selected", [(8, 1, 27026, 1), (8, 1, 48000, 1), (16, 1, 16800, 1),
                                                    (64, 8, 3300, 0), (64, 8, 5000, 1), (128, 8, 3000, 1)])
def test_short_rows_and_one_kv_head_of_selected_lists_take_no_queue(lib, hq, hkv, tokens, selected):
    blocks = -(-tokens // 64)
    assert lib.line(tokens, hq, hkv, 64, blocks, 1024, selected) >= hq * blocks


def test_the_general_line_is_three_times_the_resident_workgroups_or_twice_at_256_token_blocks(lib):
    for hq, hkv in HEADS:
        for B, resident, times in ((128, 512, 3), (256, 256, 2)):
            assert lib.line(20000, hq, hkv, B, -(-20000 // B), resident, 1) == times * resident
    assert lib.line(8100, 32, 4, 64, 127, 1024, 0) == 3 * 1024
    assert lib.line(48000, 8, 1, 64, 750, 1024, 0) == 3 * 1024


@pytest.mark.parametrize("hq,hkv", HEADS)
def test_a_batch_of_many_items_keeps_an_xcd_to_few_kv_heads(lib, hq, hkv):
    """At B = 64 and past 3072 items a batch goes by rows only where eight
    consecutive heads, an XCD's, share a KV head."""
    for n in (2000, 8000, 19070, 27244, 60000):
        order = lib.choose_batch(n, hq, hkv, 64, n // 64 + 2)
        if (n // 64 + 2) * hq > 3072 and (hq // hkv) % 8:
            assert order == BY_GROUP, n
        elif n * hq <= 3 << 18 and n * hkv <= 1 << 18:
            assert order == BY_ROW, n


@pytest.mark.parametrize("B", [64, 128, 256])
def test_few_long_rows_are_split_over_more_waves(lib, B):
    """A selection launch never leaves more than half of the 1024 SIMDs without a
    wave while a wave still scores more than 32 tokens of a long row (B = 256:
    64), and takes two waves a row of B = 128 up to 4000 rows."""
    for blocks in (1, 320, 321, 547, 1024, 2048, 4096):
        for rows in (blocks, 2 * blocks, 4 * blocks, 8 * blocks, 32 * blocks):
            t = lib.tokens_a_wave(B, blocks, rows)
            assert t in (32, 64, 128) and t <= B and (t > 32 or B < 256)
            if blocks > 320:
                assert t <= (32 if B < 256 else 64) or rows * (B // t) > 512
                assert t <= 64 or rows > 4000
