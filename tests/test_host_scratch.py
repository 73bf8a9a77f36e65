"""Register use of the built kernels: none keeps anything in scratch memory, which is what
the choices of depth by registers left (ring lengths, copy plans, staged words) are for."""
import codeobj
from paper_2008_03602_amd import _lib as L


def test_no_kernel_uses_scratch():
    res = codeobj.kernel_resources(L.LIB_PATH)
    assert len(res) > 800 and any(k.startswith("direct_f32_kernel<") for k in res)
    bad = {k: v for k, v in res.items() if v["private_segment_fixed_size"] or v["vgpr_spill_count"]}
    assert not bad, bad
