"""Which batches stream and which are tiled (use_skinny in csrc/bm_dispatch_rules.h, plain C++), and the workspaces that follow (no GPU)."""
import ctypes
import os
import subprocess

import pytest

import paper_2511_10054_amd as bm
from paper_2511_10054_amd.binding import DebugOut, LayerDesc, Weights

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
QWEN3 = dict(d=2048, E=128, F=768, K=8)
MIXTRAL = dict(d=4096, E=8, F=14336, K=2)
DEEPSEEK = dict(d=2048, E=64, F=1408, K=6, n_shared=2)

# (shape, workspace short of the fp32 output, most tokens that stream): up to 16 rows an expert on average; up to 256 rows whatever
# the number of experts; widths that the streaming kernels of multiples of 256 do not take: 16 tokens in the two-wave
# kernel while its output is small, else 16 rows; widths that the tiled kernel does not take either: up to 256 rows
LINES = [(QWEN3, 0, 256), (MIXTRAL, 0, 128), (dict(d=1024, E=16, F=1024, K=4), 0, 64), (dict(d=1024, E=16, F=1024, K=4, n_shared=1), 0, 54),
         (DEEPSEEK, 0, 16), (DEEPSEEK, 1, 2), (dict(d=8192, E=64, F=1408, K=6, n_shared=2), 0, 2), (dict(d=4096, E=64, F=1408, K=16), 0, 16),
         (dict(d=16384, E=64, F=384, K=16), 0, 15),
         (dict(d=2048, E=64, F=1376, K=6), 0, 42), (dict(d=160, E=64, F=256, K=4), 0, 64), (dict(d=192, E=64, F=128, K=4), 0, 64)]


def _desc(T, **shape):
    a = dict(T=T, d=2048, E=128, F=768, K=8, n_shared=0, R=4, H=4, dtype=bm.BM_BF16, flags=0, tae_tau=0.0, rho=0, dist_beta=0.0)
    a.update(shape)
    return LayerDesc(**a)


def test_lines_between_streaming_and_tiled_batches(tmp_path):
    """The last batch that streams and the first that is tiled, for shapes on every clause of the rule; fp32 layers never stream."""
    src = tmp_path / "rule.cpp"
    body = ""
    for shape, compact, most in LINES:
        a = dict(n_shared=0, **shape) if "n_shared" not in shape else shape
        for T, dtype, want in ((1, "BF16", 1), (most, "BF16", 1), (most + 1, "BF16", 0), (1, "F32", 0)):
            fields = " ".join("d.%s = %d;" % kv for kv in a.items())
            body += '  { bm_layer_desc d{}; d.T = %d; d.dtype = BM_%s; %s\n    if (bm::use_skinny(&d, %d) != %d) { std::printf("%s %d %s\\n"); ++bad; } }\n' % (
                T, dtype, fields, compact, want, str(a).replace('"', ""), T, dtype)
    src.write_text('#include "bm_dispatch_rules.h"\n#include <cstdio>\nint main() {\n  int bad = 0;\n' + body + '  return bad;\n}\n')
    exe = tmp_path / "rule"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2511_10054_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def _accepts(desc, nbytes):
    """bm_moe_forward takes a workspace of so many bytes (it then stops, before any launch, at the half-filled events)."""
    one = ctypes.c_void_p(256)
    w = Weights(*([256] * 8 + [0] * 5))
    dbg = DebugOut()
    dbg.stage_events[0] = 1
    rc = bm.load_library().bm_moe_forward(ctypes.byref(desc), one, ctypes.byref(w), one, one, one, one, nbytes, ctypes.byref(dbg), None)
    assert rc in (-1, -4), rc
    return rc == -1


# the next token's rows, held between the projections and the aggregation: h in bf16, o in fp32 slices of its reduction (streamed:
# whole for the Qwen3-shaped layer, two for the Mixtral-shaped one) or in bf16 (tiled).  The rest grows by
# some 100 bytes a token, each of some twenty arrays rounded up to 256.
@pytest.mark.parametrize("shape,T,o_bytes", [(QWEN3, 200, 4), (QWEN3, 255, 4), (QWEN3, 300, 2), (MIXTRAL, 100, 8), (MIXTRAL, 127, 8), (MIXTRAL, 200, 2)])
def test_batches_that_stream_keep_their_fp32_output(shape, T, o_bytes):
    n, n1 = (bm.bm_workspace_bytes(_desc(t, **shape)) for t in (T, T + 1))
    row = 2 * shape["F"] + o_bytes * shape["d"]
    assert 0 <= n1 - n - shape["K"] * row < 4096
    assert _accepts(_desc(T + 1, **shape), n1) and _accepts(_desc(T, **shape), n1)
    assert not _accepts(_desc(T + 1, **shape), n1 - 1)
