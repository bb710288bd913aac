"""Forms of the library's calls that only some sizes, layouts or launches
reach, compiled for the host against the emulation of HIP's launch API and run
under AddressSanitizer/UBSan (tests/cpu_emu/harness_forms.cpp)."""
import os
import subprocess

import pytest

from test_cpu_emulation import CLANG, CLANG_C, CSRC, EMU, ROOT


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang")
def test_forms_under_asan(tmp_path):
    fl = ["-O1", "-g", "-fsanitize=address,undefined", "-fno-omit-frame-pointer",
          "-I", EMU, "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    units = [([f"-DSU3_PREC={p}", "-x", "c++", os.path.join(CSRC, "su3_kprec.hip")], f"kp{p}.o")
             for p in range(4)]
    units += [(["-x", "c++", os.path.join(CSRC, f"su3_{k}.hip")], f"{k}.o")
              for k in ("kmisc", "kdslash", "kprog")]
    units += [([os.path.join(CSRC, f"su3_{k}.cpp")], f"{k}.o") for k in ("program", "api")]
    units += [([os.path.join(EMU, f"{k}.cpp")], f"{k}.o") for k in ("emu_globals", "harness_forms")]
    cmds = [([CLANG, "-std=c++20"] + fl + args, out) for args, out in units]
    cmds += [([CLANG_C, "-O2", "-g", "-fsanitize=address", os.path.join(ROOT, "testgen", "gen.c")],
              "gen.o"),
             ([CLANG_C, "-O2", "-g", "-ffp-contract=off", "-fsanitize=address",
               os.path.join(ROOT, "oracle", "oracle.c")], "oracle.o")]
    procs = [subprocess.Popen(cmd + ["-c", "-o", str(tmp_path / out)], stderr=subprocess.PIPE,
                              text=True) for cmd, out in cmds]
    for p in procs:
        _, err = p.communicate()
        assert p.returncode == 0, err
    exe = str(tmp_path / "harness_forms")
    subprocess.check_call([CLANG, "-fsanitize=address,undefined"] +
                          [str(tmp_path / out) for _, out in cmds] + ["-o", exe, "-lm"])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "fails 0" in r.stdout, (r.stdout + r.stderr)[-3000:]
