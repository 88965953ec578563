"""The rules that pick a scan's form (csrc/comba_rules.h), on the CPU.

They go by how many chains are at work at a time, not by how many there are: a
batch of many short or empty rows and a few long ones keeps the form that is
faster at low occupancy (the other cost it 5-20%), equal rows take the other
from 768 chains on 256 CUs."""
import os
import subprocess

import pytest

import test_scan_forms_gpu as forms

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2506_02475_amd", "csrc")
CUS = 256
MAIN = r"""
#include "comba_rules.h"
#include <cstdio>
#include <cstdlib>
int main(int, char** v) {
  long x[9];
  for (int i = 0; i < 9; ++i) x[i] = atol(v[i + 1]);
  const comba::ScanRows r{x[0], x[1], x[2], x[3]};
  const int H = x[4], dk = x[5], dv = x[6], cus = x[7];
  printf("%d %d\n", comba::scan_fwd_whole_rows(r, H, dk, dv, cus),
         comba::scan_bwd_unpadded(r, H, dk, dv, cus, x[8] != 0));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)

    def f(lens, H, dk=128, dv=128, known=True, beside=False, cus=CUS):
        ch = [-(-n // 64) for n in lens]
        args = [len(lens), sum(lens), sum(ch) if known else 0, max(ch) if known else 0, H, dk, dv,
                cus, int(beside)]
        out = subprocess.run([str(exe)] + [str(a) for a in args], capture_output=True, text=True,
                             check=True).stdout.split()
        return out[0] == "1", out[1] == "1"

    return f


def test_unequal_rows_keep_the_forms_of_few_chains(rule):
    for lens, H in (([16384] + [64] * 23, 16), ([8192] + [0] * 255, 4), ([8192] + [1] * 63, 4),
                    ([8192] * 2 + [100] * 30, 16)):
        assert len(lens) * H * 4 >= 3 * CUS  # more chains than the old line of the forward scan
        assert rule(lens, H) == (False, False), lens


def test_equal_rows_change_form_with_the_chains(rule):
    assert [rule([1024] * n, 16) for n in (4, 5, 11, 12)] == [
        (False, False), (False, True), (False, True), (True, True)]
    # beside the forward scan of the stateless backward
    assert [rule([1024] * n, 16, beside=True)[1] for n in (5, 6, 7, 8)] == [False, False, True, True]
    # dk = 256 has one form; dk = 64 one form of the reverse scan
    assert rule([1024] * 64, 16, dk=256, dv=256) == (False, False)
    assert rule([1024] * 64, 16, dk=64, dv=64) == (True, False)


def test_partly_filled_and_short_rows_keep_the_direct_forward_scan(rule):
    assert [rule([t] * 200, 4)[0] for t in (16, 70, 200, 256)] == [False, False, False, True]
    assert [rule([t] * 200, 4, dk=64, dv=64)[0] for t in (64, 256, 512)] == [False, False, True]


def test_unknown_lengths_and_unknown_devices(rule):
    assert rule([1024] * 64, 16, known=False) == (False, True)
    assert rule([1024] * 4, 16, known=False) == (False, False)
    assert rule([1024] * 64, 16, cus=0) == (False, False)


def test_the_batches_of_the_gpu_test_take_the_other_forms(rule):
    for dk, dv, T in forms.FULL:
        assert rule([T] * 64, 4 * 128 // dv, dk, dv)[0], (dk, dv, T)
    for kw in forms.PACKED:
        fwd, bwd = rule(kw["seqlens"], kw["H"], kw["dk"], kw["dv"])
        assert fwd and bwd == (kw["dk"] == 128), kw
    assert rule([191] * 64, 4) == (True, True)  # test_non_finite_values_in_every_form
    for dv, P in ((128, 8), (64, 16)):          # segments: all, and the state pass's
        assert rule([8192 // P] * P, 16, 128, dv)[1] and rule([8192 // P] * (P - 1), 16, 128, dv)[1]
