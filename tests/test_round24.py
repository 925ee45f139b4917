"""The products of a coefficient merge are rounded to the 24 bits of an fp32
value: the host build of that rounding agrees with the fp32 rounding on every
random double of the fp32 range (exact halfway cases, one in 2^29, are the
only ones that may differ), and keeps zeros, infinities and NaN.  (CPU only.)"""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2206_00470_amd", "csrc")


def test_round_to_24_bits_is_the_fp32_rounding(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC, "-o", exe,
                           os.path.join(HERE, "round24_check.cpp")])
    assert subprocess.check_output([exe], text=True).split() == ["0", "1", "1", "1", "1", "1"]
