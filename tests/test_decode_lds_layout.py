"""The LDS that the decode kernels of keys as stored ask for holds everything they address: checked on the layouts that
the kernels and their launchers are compiled with (host compiler only; no GPU is touched)."""
import os
import subprocess

import pytest

from paper_2405_03917_amd import build as cq_build

# Behind KEYS in a fused step: 2 Gh 64-bit minima; the new token's weights (one per query head of the workgroup),
# padded to 16 bytes; its record of key codes, Gh bytes and, with 10-bit codes, one word of their high bits, whose
# start is read 16 bytes at a time.
CHECK = """
#include "{source}"
namespace cq {{
template <int GH, int C, int B>
constexpr bool holds()
{{
    constexpr int D = GH * C, at = Lay<GH, B>::KEYS(D), record = at + 2 * GH * 2 + 4;
    static_assert(at % 4 == 0 && record % 4 == 0, "16-byte reads");
    static_assert(Lay<GH, B>::FLOATS(D, true) >= record + GH / 4 + (B == 10 ? 1 : 0), "the fused step's record");
    static_assert(Lay<GH, B>::FLOATS(D, true) * 4 <= 160 * 1024, "a CU's LDS");
    return true;
}}
static_assert(holds<16, 8, 8>() && holds<32, 4, 8>() && holds<64, 2, 8>() && holds<16, 8, 10>(), "");
}}
"""


@pytest.mark.parametrize("source", ["cq_decode.hip", "cq_decode_pair.hip"])
def test_a_fused_step_asks_for_the_lds_it_addresses(source, tmp_path):
    if not os.path.exists(cq_build.HIPCC):
        pytest.skip("no hipcc")
    probe = tmp_path / "layout.hip"
    probe.write_text(CHECK.format(source=source))
    cmd = [cq_build.HIPCC, *cq_build.FLAGS, "--offload-host-only", "-fsyntax-only", str(probe)]
    done = subprocess.run(cmd, capture_output=True, text=True)
    assert done.returncode == 0, done.stderr[-3000:]
