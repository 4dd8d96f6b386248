"""From how many live groups on a layer's weights go past the memory-side cache (csrc/bm_dispatch_rules.h, plain C++; no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_what_a_call_touches_decides_and_not_what_the_layer_has(tmp_path):
    """Layers on both sides of 256 MB, by the experts that are live in a call: 16 resident experts of 64 (d = F = 1024) are 101 MB
    and stay in the cache, whatever the other 48 take."""
    cases = [  # dtype, E, d, F, live groups -> streamed
        ("BM_BF16", 64, 1024, 1024, 16, 0), ("BM_BF16", 64, 1024, 1024, 42, 0), ("BM_BF16", 64, 1024, 1024, 43, 1),
        ("BM_BF16", 96, 1024, 512, 24, 0), ("BM_BF16", 128, 2048, 768, 64, 1), ("BM_BF16", 128, 2048, 768, 28, 0),
        ("BM_BF16", 8, 4096, 14336, 1, 1), ("BM_F32", 64, 1024, 512, 42, 0), ("BM_F32", 64, 1024, 512, 43, 1), ("BM_F32", 8, 65536, 65536, 1, 1)]
    src = tmp_path / "cached.cpp"
    src.write_text('#include "bm_dispatch_rules.h"\n#include <cstdio>\nint main() {\n  int bad = 0;\n' + "".join(
        '  { bm_layer_desc d{}; d.dtype = %s; d.E = %d; d.d = %d; d.F = %d;\n'
        '    if ((%d > bm::cached_groups(&d)) != %d) { std::printf("E %%d d %%d F %%d\\n", d.E, d.d, d.F); ++bad; } }\n'
        % c for c in cases) + '  return bad;\n}\n')
    exe = tmp_path / "cached"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2511_10054_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
