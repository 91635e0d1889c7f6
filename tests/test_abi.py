"""CPU checks of the C ABI: the library loads and exports every symbol that
include/mpx.h declares, and the binding covers the same set.  No compute
call is made (there is no GPU here)."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2507_03312_amd", "libmpx.so")


def declared_functions():
    src = open(os.path.join(ROOT, "include", "mpx.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    names = set(re.findall(r"\b(mpx_[a-z0-9_]+)\s*\(", src))
    return names


def test_header_declares_the_named_entry_points():
    names = declared_functions()
    for n in ["mpx_cast_to_half", "mpx_linear_fwd", "mpx_linear_bwd", "mpx_unscale_check",
              "mpx_scale_update", "mpx_adamw_masked"]:
        assert n in names


@pytest.mark.skipif(not os.path.exists(LIB), reason="libmpx.so not built")
def test_library_exports_every_declared_symbol():
    out = subprocess.run(["nm", "-D", "--defined-only", LIB], capture_output=True, text=True,
                         check=True).stdout
    exported = set(re.findall(r"\bT (mpx_[a-z0-9_]+)$", out, flags=re.M))
    missing = declared_functions() - exported
    assert not missing, missing


@pytest.mark.skipif(not os.path.exists(LIB), reason="libmpx.so not built")
def test_binding_loads_and_covers_the_header():
    from paper_2507_03312_amd import binding
    assert set(binding.EXPORTED) == declared_functions()
    # a pure host call: size queries need no device
    assert binding.mpx_linear_bwd_workspace(64, 512, 1024) > 0
    assert binding.mpx_layernorm_bwd_workspace(100, 384) > 0
    # the attention backward keeps dS on chip at every supported length
    assert all(binding.mpx_attention_bwd_workspace(64, T, 12, 64) == 0 for T in (65, 128, 129, 197, 256))


@pytest.mark.skipif(not os.path.exists(LIB), reason="libmpx.so not built")
@pytest.mark.parametrize("nk", [(2304, 768), (1152, 384), (1000, 768), (64, 64), (640, 1216)],
                         ids=lambda s: "x".join(map(str, s)))
def test_linear_bwd_workspace_never_falls_with_the_batch(nk):
    """A workspace sized for the largest batch is accepted for every smaller one."""
    from paper_2507_03312_amd import binding as mx
    sizes = [mx.mpx_linear_bwd_workspace(M, *nk) for M in range(1, 40001, 13)]
    assert sizes == sorted(sizes)


@pytest.mark.skipif(not os.path.exists(LIB), reason="libmpx.so not built")
def test_argument_checks_of_the_float32_and_fused_paths():
    """Host-side argument checks return an error before anything is
    dereferenced or launched (the pointers here are placeholders)."""
    from paper_2507_03312_amd import binding as mx
    p = 256  # never dereferenced: every call below fails its checks first
    with pytest.raises(mx.MPXError, match="bad sizes"):
        mx.mpx_layernorm_bwd(p, 2049, p, p, None, p, 2049, None, None, 4, 2049, mx.MPX_F32, None, 0,
                             None, 0)
    with pytest.raises(mx.MPXError, match="half gradients only"):
        mx.mpx_linear_bwd(p, None, p, None, 0, None, p, None, 8, 8, 8, mx.MPX_F32, p, 1 << 20, p, 0)
    with pytest.raises(mx.MPXError, match="half gradients only"):
        mx.mpx_embed_assemble_bwd(p, p, p, p, 2, 3, 8, mx.MPX_F32, p, 0)
    with pytest.raises(mx.MPXError, match="MPX_F16 or MPX_BF16"):
        mx.mpx_layernorm_fwd_cast(p, 8, p, p, p, p, None, 4, 8, mx.MPX_F32, 0)
    # the variant without a workspace rejects products whose partials exceed
    # its static array before touching the device
    M, N, K = 64, 1 << 25, 8   # 2^25 bias columns: 128 MiB of column partials
    assert mx.mpx_linear_bwd_workspace(M, N, K) > mx.MPX_LINEAR_BWD_NOALLOC_SCRATCH
    with pytest.raises(mx.MPXError, match="static scratch"):
        mx.mpx_linear_bwd_noalloc(p, p, p, None, 0, None, p, p, M, N, K, mx.MPX_BF16, None, 0)
    with pytest.raises(mx.MPXError, match="M, N, K"):
        mx.mpx_linear_bwd_noalloc(p, p, p, None, 0, None, p, p, 0, N, K, mx.MPX_BF16, None, 0)
    with pytest.raises(mx.MPXError, match="MPX_F16, MPX_BF16 or MPX_F32"):
        mx.mpx_linear_fwd(p, p, None, None, p, None, 8, 8, 8, 7, 0, 0)
