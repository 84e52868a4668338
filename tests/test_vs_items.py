"""The token-level rows' items on the CPU: the plain C++ of csrc/vs_items.h compiled with g++, undefined behaviour an error."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2505_19578_amd", "csrc")


def _compile_and_run(tmp_path, body):
    src, exe = tmp_path / "t.cc", tmp_path / "t"
    src.write_text('#include "vs_items.h"\n#include <cstdio>\nint main() {\n' + body + "\nreturn 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I" + CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr + r.stdout
    return r.stdout


# the longest prompt has 2^16 tiles; mask_pre goes on with 64 x + 96 - 63
@pytest.mark.parametrize("first", [0, 1, 63, 65534])
def test_tile_distance_is_defined_for_every_item(tmp_path, first):
    out = _compile_and_run(tmp_path, f"""
      const int first = {first};
      for (int g = 0; g < 65536; ++g) {{
        volatile int start = 64 * vs_tiles_below(first, VS_GATHERED | (uint32_t)g) + 96 - 63;
        (void)start;
        if (g <= first + 1 && vs_tiles_below(first, (uint32_t)g) != first - g) return 1;
      }}
      std::puts("ok");""")
    assert out == "ok\n"
