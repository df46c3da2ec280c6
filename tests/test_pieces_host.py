"""The launches that many agents or points are cut into, checked on the CPU by
tests/cpp/pieces_check.cpp under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pieces_cover_every_item_once(tmp_path):
    exe = str(tmp_path / "pieces_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
                    "-Wextra", "-I" + os.path.join(ROOT, "paper_1904_01201_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "pieces_check.cpp"), "-o", exe], check=True, timeout=120)
    assert subprocess.run([exe], capture_output=True, text=True, timeout=120).stdout.strip() == "ok"
