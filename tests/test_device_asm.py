"""What the compiler does not look for inside inline assembly, checked in the
assembly that it emits for it (no GPU needed)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_08342_amd", "csrc")


def test_direct_lds_loads_wait_for_m0(tmp_path):
    """A load into LDS needs a wait state after a scalar write of M0 (its LDS
    address): some instruction stands between the two.  Only the helper in
    device.h writes such loads."""
    from paper_2509_08342_amd import build as b
    src = tmp_path / "probe.hip"
    src.write_text('#include "device.h"\n'
                   "__global__ void probe(const unsigned char* p, uint32_t a) {\n"
                   "  msk::lds_load16(p + 16 * threadIdx.x, a);\n"
                   "  msk::lds_load16(p + 16 * threadIdx.x + 1024, a + 1024);\n"
                   "  msk::wait_vm<0>();\n"
                   "}\n")
    text = subprocess.run([b.HIPCC, *b.FLAGS, "-I" + CSRC, "--offload-device-only", "-S", str(src), "-o", "-"],
                          check=True, capture_output=True, text=True).stdout
    ops = [l.strip() for l in text.splitlines() if re.match(r"\s+[a-z]+_[a-z0-9_]+(\s|$)", l)]
    loads = [i for i, l in enumerate(ops) if l.startswith("global_load_lds")]
    assert len(loads) == 2
    for i in loads:
        assert not re.match(r"s_\w+ m0\b", ops[i - 1]), ops[i - 2:i + 1]
    for name in os.listdir(CSRC):
        if name != "device.h":
            assert not re.search(r'^\s*"[^"]*load_lds', open(os.path.join(CSRC, name)).read(), re.M), name
