"""The short sequences of the straight cells (drift, curvature, radiation step,
logarithm, deviate, and the quotient with a rounded reciprocal) on the CPU, from
the device header itself, with the hardware estimates modelled at their measured
error bounds: wherever a step does not hand its operands over to the general
operations, it gives the general operations' bits."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(os.path.dirname(HERE), "paper_2310_00317_amd", "csrc", "xtm_maps.h")
CLANG = "/opt/rocm/llvm/bin/clang++"


def _bodies(text):
    """The header with the IEEE operations instead of the short sequences."""
    def body(signature, code):
        nonlocal text
        at = text.index(signature)
        start, end = text.index("{", at), text.index("\n}", at)
        text = text[:start] + "{ " + code + text[end:]
    body("double sqrt_in(double x, double& h_out)", "h_out = 0.5 / sqrt(x); return sqrt(x);")
    body("double div_by_root(double a, double root, double h)", "return a / root;")
    body("double div_in(double a, double b)", "return a / b;")
    body("double div_known(double a, double b, double r)", "return a / b;")
    return text


def test_short_sequences_give_the_general_bits(tmp_path):
    with open(HEADER) as f:
        text = f.read()
    text = re.sub(r"\basm\b[^;]*;", ";", text.replace("#pragma once", ""))
    assert "asm(" not in text
    defines = "".join(f"#undef {m}\n" for m in re.findall(r"#define (\w+)", text))
    (tmp_path / "short.h").write_text(text + defines)
    (tmp_path / "generic.h").write_text(_bodies(text).replace("namespace xtmm", "namespace generic"))
    exe = str(tmp_path / "short_sequences")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-fno-fast-math", "-mfma", "-w",
                    "-I", str(tmp_path), "-o", exe,
                    os.path.join(HERE, "cpu_emulation", "short_sequences.cpp"), "-lm"], check=True)
    n = 2000000
    out = subprocess.run([exe, str(n)], check=True, capture_output=True, text=True).stdout
    rows = re.findall(r"^(.*) served (\d+) wrong (\d+)$", out, re.M)
    assert len(rows) == 11, out
    for what, served, wrong in rows:
        assert int(wrong) == 0, out
        assert int(served) >= n // 10, out
