"""What the compiler makes of a kernel where the source alone does not show it: the gfx950 assembly of one instance."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2601_01712_amd import build

CSRC = os.path.join(os.path.dirname(os.path.abspath(build.__file__)), "csrc")


def assembly(tmp_path, header, instance):
    hipcc = next((p for p in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc") if p and os.path.exists(p)), None)
    if hipcc is None:
        pytest.skip("no hipcc")
    src, out = tmp_path / "one.hip", tmp_path / "one.asm"
    src.write_text(f'#include "{os.path.join(CSRC, header)}"\nusing namespace relaygr;\ntemplate __global__ void {instance};\n')
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


@pytest.mark.parametrize("dh,pieces", [(32, 2), (64, 4), (128, 8)])
def test_attention_tiles_take_one_lds_address_per_four_pieces(tmp_path, dh, pieces):
    """A wavefront moves `pieces` of 1 KiB of every key tile; all but every fourth take their place from the immediate offset."""
    text = assembly(tmp_path, "attention.h", f"relaygr::attn_bf16_kernel<Bf16, {dh}, 1, 4, false, 1>(AttnParams)")
    loads = re.findall(r"^\s+buffer_load_dwordx4 .*\blds$", text, re.M)
    own = [ld for ld in loads if "offset:" not in ld]
    assert loads and len(loads) % pieces == 0
    assert len(own) == len(loads) // pieces * ((pieces + 3) // 4)


@pytest.mark.parametrize("instance", ["64, 1, 4, false, 1", "64, 2, 4, false, 2", "128, 1, 8, true, 1"])
def test_attention_reads_its_work_item_by_scalar_loads(tmp_path, instance):
    """A field narrower than a word takes a vector load, a round trip to memory that the loads of the candidates' own keys wait for; and the rows' own
    chunks are 32-bit offsets from scalar bases."""
    text = assembly(tmp_path, "attention.h", f"relaygr::attn_bf16_kernel<Bf16, {instance}>(AttnParams)")
    start = text[:text.index("s_barrier")]
    assert not re.search(r"global_load_(u|s)(byte|short)", start)
    assert re.search(r"global_load_dwordx4 v\[\d+:\d+\], v\d+, s\[", start)
