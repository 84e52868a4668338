"""The token-level rows' items on the CPU: the plain C++ of csrc/vs_items.h compiled with g++, undefined behaviour an error."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2505_19578_amd", "csrc")


def _compile_and_run(tmp_path, body):
    src, exe = tmp_path / "t.cc", tmp_path / "t"
    src.write_text('#include "vs_items.h"\n#include <cstdio>\n#include <initializer_list>\nint main() {\n' + body + "\nreturn 0;\n}\n")
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


@pytest.mark.parametrize("block", [64, 128])
@pytest.mark.parametrize("maps", [1, 2, 3, 32, 128, 256])
def test_rows_split_into_launches(tmp_path, block, maps):
    """The launches partition the rows, a launch's items fit the room, and the first row of the next would not have fitted.  One
    launch up to a block or two below 32 block^2 tokens, two from there on; never without room for a row."""
    out = _compile_and_run(tmp_path, f"""
      const int block = {block}, spb = block / 64;
      const size_t maps = {maps};
      auto launches = [&](int nqb) {{
        const int64_t room = vs_item_room(maps, (size_t)nqb * block, block);
        if (vs_band_bytes(maps, (size_t)nqb * block) + maps * room * sizeof(VsItem) > vs_statistics_bytes(maps, (size_t)nqb * block, block)) return -1;
        int n = 0;
        for (int row1 = nqb, row0; row1 > 0; row1 = row0, ++n) {{
          row0 = vs_first_row(row1, room, spb);
          int64_t items = 0;
          for (int r = row0; r < row1; ++r) {{
            if (items != vs_items_before(r, row0, spb)) return -2;
            items += (int64_t)spb * (r + 1);
          }}
          if (row0 == row1 || items > room) return -3;
          if (row0 > 0 && items + (int64_t)spb * row0 <= room) return -4;
        }}
        return n;
      }};
      for (int nqb : {{1, 2, 3, 64, 1000, 32 * block - 2}}) if (launches(nqb) != 1) return 1;
      std::printf("%d\\n", launches(32 * block - 1));
      for (int nqb : {{32 * block, 32 * block + 1, 48 * block}}) if (launches(nqb) != 2) return 2;
      if (launches(32768) < 2) return 3;""")
    # the bitmaps take 32 (block 64) or 128 (block 128) items of a head, the numbers per query leave 32 or 64
    assert int(out) == (1 if block == 64 else 2)
