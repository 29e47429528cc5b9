"""Whether a pass exceeds the memory-side cache goes by the keys it reads and not by the room there is for them."""
import os
import subprocess

import pytest

from paper_2505_21467_amd import build

SOURCE = r"""
#include <stdio.h>
#include <stdlib.h>
#include "fc_internal.h"
int main(int argc, char **argv)
{
    fc_config c = {};
    c.n_layers = atoi(argv[1]);
    c.batch = 1;
    c.hidden = 3584;
    c.n_q_heads = 28;
    c.n_kv_heads = 4;
    c.head_dim = 128;
    c.max_seq = atoi(argv[2]);
    c.dtype = FC_BF16;
    printf("%d", (int)fc_read_once(fc_pass_bytes(c, atoi(argv[4]), atoi(argv[3]))));
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("read_once")
    (d / "main.cpp").write_text(SOURCE)
    subprocess.run([build.HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                    str(d / "main.cpp"), "-o", str(d / "main")], check=True, capture_output=True, timeout=120)
    return str(d / "main")


@pytest.mark.parametrize("layers,max_seq,keys,d_ff,once", [
    (1, 1056, 1056, 0, 0), (1, 131072, 1056, 0, 0), (1, 131072, 131072, 0, 1), (2, 131072, 1056, 0, 0), (2, 131072, 65536, 0, 1),
    (8, 1056, 1056, 0, 1), (1, 1056, 1056, 18944, 1),
])
def test_keys_that_are_read_count(program, layers, max_seq, keys, d_ff, once):
    out = subprocess.run([program, str(layers), str(max_seq), str(keys), str(d_ff)], check=True, capture_output=True, text=True, timeout=60)
    assert out.stdout == str(once)
