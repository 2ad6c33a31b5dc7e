"""The rules that choose between forms of a kernel (csrc/dispatch.h), compiled for the host and asked at the sizes on either side of their lines."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_06040_amd", "csrc")
SOURCE = """
#include "dispatch.h"
using namespace br;
extern "C" {
int tile_output_streams(unsigned long long bytes) { return rule::tile_output_streams(bytes); }
int persistent_output_stays(unsigned long long bytes, int K, int gelu) { return rule::persistent_output_stays(bytes, K, gelu); }
int attention_parts(int dh, int brief, long long left, long long whole, int units) { return rule::attention_parts(dh, brief, left, whole, units); }
int attention_pair(int tokens, long long tiles128, long long tiles256, int units) { return rule::attention_pair(tokens, tiles128, tiles256, units); }
int weights_stay(double bytes) { return rule::weights_stay(bytes); }
int read_ahead(unsigned long long room, unsigned long long bytes) { return rule::read_ahead(room, bytes); }
int f32_small(int M, int N, int units) { return rule::f32_small(M, N, units); }
void f32_ring_tile(int M, int N, int K, int rps, int units, int* rb, int* cb) { rule::f32_ring_tile(M, N, K, rps, units, rb, cb); }
}
"""
CU = 256


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "rules.so"), str(d / "rules.cpp")], check=True)
    return C.CDLL(str(d / "rules.so"))


def test_large_outputs_of_the_tile_kernels_go_past_the_caches(rule):
    """hidden 960 and 2880, whose products the persistent kernel does not take: first MLP layer of 8 and of 64 samples of 1101 rows, QKV of 64."""
    stream = lambda M, N: bool(rule.tile_output_streams(C.c_ulonglong(M * N * 2)))
    assert not stream(8 * 1101, 4 * 960) and not stream(4 * 1101, 4 * 2880)
    assert stream(64 * 1101, 4 * 960) and stream(64 * 1101, 3 * 2880)
    assert not stream(40960, 2048) and stream(40961, 2048)


def test_outputs_of_the_persistent_kernel_that_stay_in_the_caches(rule):
    """First MLP layers that plain stores cost 2 to 7 % of a velocity call, and ones that they gain 1 to 5 % for; QKV rows, which have a line of their own."""
    fc1 = lambda rows, H: bool(rule.persistent_output_stays(C.c_ulonglong(rows * 4 * H * 2), H, 1))
    qkv = lambda rows, H: bool(rule.persistent_output_stays(C.c_ulonglong(rows * 3 * H * 2), H, 0))
    for H, rows in ((256, 53 * 1101), (512, 27 * 1101), (512, 315 * 93), (512, 378 * 93), (768, 18 * 1101), (768, 168 * 93), (1024, 11 * 1101),
                    (1024, 13 * 1101), (1024, 158 * 93)):
        assert not fc1(rows, H) and qkv(rows, H), (H, rows)
    for H, rows in ((256, 441 * 93), (512, 126 * 93), (512, 221 * 93), (768, 63 * 93), (1024, 8 * 1101), (1024, 47 * 93), (1536, 105 * 93), (2048, 8 * 1101), (3072, 3 * 1101)):
        assert fc1(rows, H), (H, rows)
    assert qkv(16 * 1101, 1024) and not qkv(19 * 1101, 1024) and not qkv(441 * 93, 1024) and qkv(16 * 1101, 1536) and not qkv(22 * 1101, 2304)
    assert not fc1(2047, 1024 * 2) and fc1(2048, 1024 * 2) and not qkv(11 * 93, 3072)


def test_attention_cuts_the_tiles_of_a_last_round_that_leaves_units_idle(rule):
    """Never into more workgroups than units at head dim 128 (but for those that are whole); all units or those of one compute die."""
    parts = lambda dh, left, whole, units=CU, brief=0: rule.attention_parts(dh, brief, C.c_longlong(left), C.c_longlong(whole), units)
    for units in (CU, CU // 8):
        for left in range(units + 1):
            p = parts(128, left, 7 * units, units)
            assert p in (1, 2, 4) and (p == 1 or left * p <= units) and (p > 1) == (2 * left <= units) and p == parts(128, left, 0, units)
            assert parts(64, left, 3 * units, units) == 1 and parts(64, left, 0, units) == (2 if 5 * left <= 3 * units else 1)
        # two parts of every tile, three workgroups a unit: as many as start at once
        assert all(parts(64, left, 0, units) == (2 if 2 * left <= 3 * units else 1) for left in range(units + 1, 3 * units))


def test_attention_in_two_workgroups_a_unit(rule):
    """Sizes that one workgroup of 256 queries a unit cost 7 to 60 %, and ones that two of 128 cost 3 to 30 %; pairs are dealt out by die from 32 on."""
    def pair(L, pairs):
        dies = 8 if pairs >= 32 else 1
        tiles = lambda rows: C.c_longlong((-(-pairs // 8) if dies == 8 else pairs) * -(-L // rows))
        return bool(rule.attention_pair(L, tiles(128), tiles(256), CU // dies))
    for L, pairs in ((129, 144), (192, 96), (192, 1536), (193, 288), (257, 144), (257, 768), (320, 48), (513, 48), (640, 96), (800, 144), (1024, 72), (1024, 192), (1101, 56), (1101, 72), (1101, 192),
                     (1500, 56), (2048, 48), (2048, 384), (4608, 6)):
        assert pair(L, pairs), (L, pairs)
    for L, pairs in ((1, 1536), (65, 288), (128, 384), (128, 1536), (129, 64), (192, 48), (193, 144), (193, 192), (257, 40), (385, 24), (513, 24), (800, 40), (1101, 6), (1101, 40), (1101, 64), (1500, 48), (2048, 24), (2048, 40),
                     (2049, 384), (2300, 48), (3000, 96),
                     (4608, 24), (8192, 6), (8192, 48), (33272, 12)):
        assert not pair(L, pairs), (L, pairs)


def test_weights_are_read_ahead_where_a_good_part_of_them_fits(rule):
    """A block's four matrices (2 x 12 H^2 bytes) against what the idle units read during an attention of L tokens: 2 MB a tile of 64 keys, and four
    tiles' time around them, of 256 units."""
    def ahead(H, head_dim, L, B):
        idle = (CU - B * (H // head_dim) * -(-L // 128)) // 8 * 8
        return idle >= 32 and bool(rule.read_ahead(C.c_ulonglong(2 ** 21 * (-(-L // 64) + 4) // 256 * idle), C.c_ulonglong(24 * H * H)))
    for case in ((1024, 64, 1101, 1), (1024, 128, 333, 2), (1024, 64, 100, 1), (1536, 128, 1101, 1), (2048, 64, 200, 2), (2560, 128, 613, 1)):
        assert ahead(*case), case
    for case in ((3072, 128, 333, 1), (3072, 128, 80, 1), (3072, 128, 1101, 1), (2880, 64, 200, 1), (2560, 64, 333, 1), (2560, 128, 613, 2), (1024, 64, 1101, 2)):
        assert not ahead(*case), case


def test_weights_that_stay_in_the_cache_are_not_read_ahead(rule):
    """12 matrices of H^2 a block, 6 of modulation and 2 at the end: networks that lost 2 % by it, and ones that gain 3 to 9 %."""
    stay = lambda H, blocks: bool(rule.weights_stay(C.c_double((18.0 * blocks + 2) * H * H * 2)))
    assert stay(768, 9) and stay(768, 11) and stay(1024, 5) and stay(1024, 6) and stay(512, 24)
    assert not stay(768, 13) and not stay(1024, 7) and not stay(1024, 12) and not stay(512, 37) and not stay(1536, 3) and not stay(3072, 24)


def test_fp32_products_small_tiles_or_which_ring_tile(rule):
    """The rule is a function of sizes and the number of units alone (a caller that asked the runtime for them once a tile paid 1.3 us a call)."""
    def tile(M, N, K, rps=0):
        rb, cb = C.c_int(), C.c_int()
        rule.f32_ring_tile(M, N, K, rps, CU, C.byref(rb), C.byref(cb))
        return rb.value, cb.value
    small = lambda M, N: bool(rule.f32_small(M, N, CU))
    assert small(599, 768) and small(24 * 32, 32 * 32) and not small(24 * 32 + 1, 32 * 32) and not small(1101, 1024) and not small(1624, 768)
    assert not small(2 ** 31 - 1, 1024)
    # one round of 144 x 128 tiles (0.97 full) for 4404 x 1024; two of 128 x 128 for 32 of the same rows
    assert tile(4404, 1024, 4096) == (9, 2)
    for M, N, K in ((1101, 1024, 4096), (1624, 768, 3072), (2000, 1536, 512), (32768, 4096, 4096)):
        rb, cb = tile(M, N, K)
        rounds = lambda r, c: -(-(-(-M // (16 * r)) * -(-N // (64 * c))) // CU)
        # no other tile needs less of the matrix pipes by a quarter
        assert all(rounds(rb, cb) * rb * cb <= 1.25 * rounds(r, c) * r * c for r in range(2, 13) for c in (1, 2)), (M, N, K)
    # gated residual: no taller than a sample, unless that is shorter than the lowest tile
    for rps in (7, 31, 32, 50, 100, 191, 192):
        rb, cb = tile(rps * 300, 1024, 1024, rps)
        assert rb == 2 or 16 * rb <= rps, rps
