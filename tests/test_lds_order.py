"""The one place where lanes exchange values through LDS (the accumulator's stores of the reduction) tells the
compiler the order of writes and reads: checked in the library's own LLVM IR, because a build that happens to
keep the order gives the right results without it."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lds_writes_and_reads_are_ordered_for_the_compiler(tmp_path):
    spec = importlib.util.spec_from_file_location("lib_build", os.path.join(ROOT, "paper_2205_00119_amd", "build.py"))
    lib_build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(lib_build)
    if not os.path.exists(lib_build.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "kernels.ll")
    flags = [f for f in lib_build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([lib_build.HIPCC, *flags, "--offload-device-only", "-S", "-emit-llvm", "-o", out,
                    os.path.join(ROOT, "paper_2205_00119_amd", "csrc", "kernels.hip")], check=True, capture_output=True)
    kernels, accesses = {}, None
    for line in open(out):
        start = re.match(r"define .*@(\S+?)\(", line)
        if start:
            accesses = kernels.setdefault(start.group(1), [])
        elif re.match(r'\s+fence syncscope\("wavefront"\) (release|acquire)', line):
            accesses.append("|")
        elif re.match(r"\s+store .*ptr addrspace\(3\)", line):
            accesses.append("w")
        elif re.match(r"\s+%\S+ = load .*ptr addrspace\(3\)", line):
            accesses.append("r")
    with_lds = {name: re.sub(r"\|+", "|", "".join(a)) for name, a in kernels.items() if "w" in a or "r" in a}
    assert with_lds and all("rsa" in name for name in with_lds)
    # two writes, then two reads in the order of the store, then whatever the next pass writes
    for name, order in with_lds.items():
        assert re.fullmatch(r"(w+\|r+\|)+", order), (name, order)
