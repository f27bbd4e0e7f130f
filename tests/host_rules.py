"""Compiles a host-only header of the library with a small program around it, for tests of
the arithmetic that it holds (no GPU, no HIP)."""
import os
import subprocess

from paper_2608_07814_amd import build as B


def run_program(tmp_path, header, body, lines):
    """`body` is the statements of a loop that reads one line's numbers from
    std::cin and prints one line; returns the printed rows as lists of text."""
    src = tmp_path / "program.cpp"
    exe = str(tmp_path / "program")
    src.write_text('#include <cmath>\n#include <cstdio>\n#include <iostream>\n#include "%s"\n'
                   "int main() {\n  while (std::cin >> std::ws, !std::cin.eof()) {\n%s\n  }\n}\n" % (header, body))
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", B.CSRC, str(src), "-o", exe], check=True)
    out = subprocess.run([exe], input="\n".join(" ".join(str(v) for v in row) for row in lines), text=True,
                         stdout=subprocess.PIPE, check=True).stdout
    rows = [r.split() for r in out.splitlines()]
    assert len(rows) == len(lines)
    return rows
