"""CPU-side checks of the rules that choose kernels, block orders and packings: host functions of the library, called by
their C++ names, compared with what they claim over the sizes they accept."""
import ctypes
import os
import re
import subprocess

import pytest

import paper_2510_26527_amd as psd


@pytest.fixture(scope="module")
def rule():
    """rule(name, restype, *argtypes): the library's host function psd::name."""
    if not os.path.exists(psd.LIB_PATH):
        from paper_2510_26527_amd import build
        build.build()
    lib = psd.lib()
    syms = subprocess.run(["nm", "-D", "--defined-only", psd.LIB_PATH], check=True, capture_output=True, text=True).stdout.split()

    def find(name, restype, *argtypes):
        f = getattr(lib, next(s for s in syms if re.match(rf"_ZN3psd{len(name)}{name}E", s)))
        f.restype, f.argtypes = restype, argtypes
        return f
    return find


class ChunkOrder(ctypes.Structure):
    _fields_ = [("heads_inner", ctypes.c_uint32), ("chunk", ctypes.c_uint8 * 32)]


@pytest.mark.parametrize("group", [1, 2, 3, 4, 7, 8, 16, 32, 64])
def test_attention_chunks_go_out_longest_first(rule, group):
    """Every chunk of 128 query rows once, in the order of the keys it sees: the position of its last row, counted row by row."""
    order = rule("attn_chunk_order", ChunkOrder, ctypes.c_int, ctypes.c_int, ctypes.c_int)
    for R in range(max(1, 65 // group), 4096 // group + 1, 1 if group > 16 else 7):
        rows = [i % R for i in range(group * R)]
        seen = [max(rows[c:c + 128]) for c in range(0, group * R, 128)]
        o = order(R, group, 128)
        chunks = list(o.chunk[:len(seen)])
        assert o.heads_inner == 1 and sorted(chunks) == list(range(len(seen))), (R, group)
        assert all(seen[a] >= seen[b] for a, b in zip(chunks, chunks[1:])), (R, group, chunks)


@pytest.mark.parametrize("B,R,h_kv,d_h,keys,longest", [
    (16, 1000, 16, 128, 1000, True), (8, 500, 32, 128, 1000, True), (16, 1000, 32, 128, 2000, True), (16, 1000, 8, 128, 5000, True), (2, 700, 32, 128, 4700, True),
    (32, 40, 8, 128, 4040, False), (8, 200, 32, 128, 1200, False), (32, 200, 16, 128, 1200, False), (32, 500, 8, 128, 2500, False)])
def test_attention_order_by_the_bytes_between_a_heads_chunks(rule, B, R, h_kv, d_h, keys, longest):
    """On each side of the line: batches measured to be faster longest first, and with each head's blocks side by side."""
    assert rule("attn_longest_first", ctypes.c_bool, *[ctypes.c_int] * 5)(B, R, h_kv, d_h, keys) == longest


@pytest.mark.parametrize("d_model,d_ffn,by_tiles", [
    (6656, 17920, False), (8192, 16896, False), (6656, 4096, False), (5120, 128, False),
    (3584, 18944, True), (4096, 14336, True), (8192, 28672, True), (5120, 27648, True), (4096, 16896, True)])
def test_4bit_gate_up_by_tiles_where_they_fill_the_chip(rule, d_model, d_ffn, by_tiles):
    """On each side of the line: widths measured to be faster in equal ranges of K, with a SwiGLU launch, and by tiles."""
    assert rule("gemm_w4_gates", ctypes.c_bool, ctypes.c_int, ctypes.c_int)(d_model, d_ffn) == by_tiles


@pytest.mark.parametrize("B,R,h_q,h_kv,d_h,keys,splits", [
    (1, 256, 32, 8, 128, 512, 2), (1, 293, 28, 4, 128, 512, 2), (1, 205, 40, 8, 128, 512, 2), (1, 512, 16, 16, 64, 512, 2), (2, 257, 16, 16, 64, 449, 2),
    (2, 129, 32, 8, 128, 512, 1), (1, 258, 32, 32, 128, 258, 1), (3, 150, 32, 8, 128, 510, 1), (2, 257, 16, 16, 64, 448, 1), (2, 256, 32, 8, 64, 512, 1),
    (2, 256, 32, 8, 64, 513, 2), (1, 200, 32, 32, 128, 500, 2)])
def test_short_prompts_keep_two_splits_where_one_leaves_cus_idle(rule, B, R, h_q, h_kv, d_h, keys, splits):
    """Up to 512 keys in one split: 8192 rows x heads and 80 blocks of 128 query rows; of 64-wide heads 128 blocks, or up to 448 keys."""
    pick = rule("attn_pick_splits", ctypes.c_int, *[ctypes.c_int] * 7, ctypes.c_bool)
    assert pick(psd.PSD_BF16, B, R, h_q, h_kv, d_h, keys, False) == splits


class GemmBands(ctypes.Structure):
    _fields_ = [("strips", ctypes.c_int), ("paired", ctypes.c_int), ("inverse", ctypes.c_uint32), ("owned", ctypes.c_bool)]


def test_bands_are_of_the_widths_that_are_built(rule):
    """Every width of a model: gate|up in whole bands of 1 to 7 strips of each matrix, QKV in bands of 3 to 6 or on shared 64-row tiles; and the
    band of a strip as the kernels find it, by the inverse of the width."""
    gate = rule("gemm_gate_bands", GemmBands, ctypes.c_int)
    qkv = rule("gemm_qkv_bands", GemmBands, ctypes.POINTER(ctypes.c_int))
    def band(b, strip):
        return strip if b.strips == 1 else strip * b.inverse >> 32
    for n in range(64, 64 * 1024, 64):
        b = gate(n)
        assert b.owned and 1 <= b.strips <= 7 and b.paired == -(-n // (16 * b.strips)), n
        assert all(band(b, s) == s // b.strips for s in {0, b.strips - 1, b.strips, n // 16 - 1}), n
        b = qkv((ctypes.c_int * 3)(n, 64, 64))
        assert not b.paired and (3 <= b.strips <= 6 if b.owned else b.strips == 4), n
        assert all(band(b, s) == s // b.strips for s in {0, b.strips - 1, b.strips, n // 16 + 7}), n


class RowsPlan(ctypes.Structure):
    _fields_ = [("used", ctypes.c_bool), ("whole", ctypes.c_bool), ("waves", ctypes.c_int), ("tiles", ctypes.c_int), ("blocks", ctypes.c_int),
                ("slots", ctypes.c_int)]


@pytest.mark.parametrize("d_model,hq,hk,d_head,strips,rows", [
    (4096, 32, 32, 128, 3, "shared"), (3840, 44, 22, 128, 3, "shared"), (2944, 58, 29, 128, 4, "shared"), (2176, 78, 39, 128, 5, "shared"),
    (1792, 64, 64, 128, 6, "shared"), (640, 64, 64, 128, 6, "no"), (512, 60, 60, 128, 6, "whole"), (128, 44, 22, 128, 3, "no"), (256, 64, 32, 128, 4, "no"), (128, 80, 40, 128, 5, "no"), (4224, 66, 66, 64, 0, "shared")])
def test_qkv_bands_and_who_reads_them(rule, d_model, hq, hk, d_head, strips, rows):
    """What the GPU tests of the band kernel and of the rows kernel take their sizes for: the width of the QKV bands (0: shared 64-row tiles, not
    bands), and whether 17 to 64 rows read them in shared tiles, in whole ones, or not (the tiled kernel on the row-major weights)."""
    n = (ctypes.c_int * 3)(hq * d_head, hk * d_head, hk * d_head)
    b = rule("gemm_qkv_bands", GemmBands, ctypes.POINTER(ctypes.c_int))(n)
    assert (b.strips if b.owned else 0) == strips
    plan = rule("gemm_rows_plan", RowsPlan, ctypes.c_int, ctypes.c_int, ctypes.POINTER(ctypes.c_int), ctypes.c_int, ctypes.c_bool)
    for M in (17, 45, 64):
        p = plan(M, d_model, n, 3, False)
        assert ("whole" if p.whole else "shared" if p.used else "no") == rows, M
