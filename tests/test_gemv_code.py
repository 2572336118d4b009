"""What the compiler makes of the batch-1 kernels.  They run at the largest register count that leaves four wavefronts per SIMD, so that
a change of a prologue shows as spills in the streaming loop, which no test of results notices."""
import os
import re
import subprocess

import pytest

from paper_2605_26092_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """gfx950 assembly of goq_gemv.hip, compiled as the library is."""
    out = str(tmp_path_factory.mktemp("code") / "goq_gemv.s")
    name = "goq_gemv.hip"
    subprocess.run(["hipcc", "-S", "--offload-device-only"] + [f for f in build.FLAGS if f != "-shared"] + build.EXTRA[name]
                   + ["-o", out, os.path.join(build.CSRC, name)], check=True, stderr=subprocess.DEVNULL)
    return open(out).read()


def test_no_vector_register_is_spilled(assembly):
    kernels = re.findall(r"\.name:\s+(\S*gemv_\S*kernel\S*)\n.*?\.vgpr_spill_count:\s+(\d+)", assembly, re.S)
    assert len(kernels) == 26                          # streaming: 2 widths x 5 activation types x 2 forms; 6 for small layers
    assert not [k for k in kernels if int(k[1])]


def test_first_weights_are_requested_while_activations_are_on_their_way(assembly):
    """From the request of the first activations to that of the first weights (the non-temporal loads) nothing waits for the
    activations, whatever has to be done to their bits afterwards."""
    late, kernels = [], re.findall(r"^(_Z\S*gemv_(?:stream_|rows_)?kernel\S*):(.*?)s_endpgm", assembly, re.S | re.M)
    assert len(kernels) == 26
    for name, body in kernels:
        loads = list(re.finditer(r"global_load_\S+.*", body))
        first = next(i for i, m in enumerate(loads) if m.group(0).split(";")[0].rstrip().endswith(" nt"))
        if "s_waitcnt vmcnt(" in body[loads[first - 1].end():loads[first].start()]:
            late.append(name)
    assert not late
