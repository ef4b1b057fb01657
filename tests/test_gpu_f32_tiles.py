"""The tests of fp32 inputs once more on the kernel with 128-row tiles: their sizes are small enough for the kernel that deals the
keys to the waves, unless a flag asks for tiles (NO_F16, which changes nothing in that kernel)."""
import pytest

from paper_2510_08431_amd import binding
from test_gpu_f32_ranges import *          # noqa: F401,F403
from test_gpu_mfma_f32 import *            # noqa: F401,F403

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def tile_kernel(monkeypatch):
    call = binding.attn_jvp_fwd_ex
    monkeypatch.setattr(binding, "attn_jvp_fwd_ex", lambda *a, **kw: call(*a, **{**kw, "flags": kw.get("flags", 0) | binding.FLAG_NO_F16}))
