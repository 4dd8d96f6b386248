"""Which co-activation batches are counted in short chunks (csrc/bm_dispatch_rules.h, plain C++; no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_short_chunks_only_where_they_were_measured_faster(tmp_path):
    """Batches on both sides of the line: 8192 tokens of 8 out of 256 experts take 14.5 us in short chunks and 12.1 in long ones."""
    cases = [  # tokens, slots, experts -> short
        ((8192, 8, 256), 0), ((8192, 8, 128), 0), ((16384, 8, 64), 0), ((32768, 2, 16), 0), ((4096, 4, 64), 0), ((8192, 6, 256), 0),
        ((2048, 8, 256), 1), ((4096, 8, 128), 1), ((8192, 8, 64), 1), ((32768, 8, 16), 1), ((16384, 2, 16), 1), ((1000, 1, 256), 1)]
    src = tmp_path / "coact.cpp"
    src.write_text('#include "bm_dispatch_rules.h"\n#include <cstdio>\nint main() {\n  int bad = 0;\n' + "".join(
        '  if (bm::coact_short_chunks(%d, %d, %d) != %d) { std::printf("%d %d %d\\n"); ++bad; }\n' % (*c, want, *c) for c, want in cases) +
        '  return bad;\n}\n')
    exe = tmp_path / "coact"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2511_10054_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
