"""The C-ABI library loads and exports every function that include/bitlinear.h declares.
No compute call is made (no GPU needed); size queries and argument validation run on the host."""
import ctypes
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "bitlinear.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"\b([a-z_0-9]+)\s*\([^;{}]*\)\s*;", text)
    return sorted(set(names))


@pytest.fixture(scope="module")
def lib():
    from paper_2411_04965_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build(verbose=False)
    return binding.lib()


def test_header_lists_the_four_entry_points():
    names = declared_functions()
    for must in ("bitlinear_a4", "bitlinear_a8_sparse", "quantize_act", "pack_ternary"):
        assert must in names


def test_every_declared_symbol_is_exported(lib):
    from paper_2411_04965_amd import binding
    for name in declared_functions():
        assert hasattr(lib, name), name
        assert name in binding._SIGNATURES, "binding lacks " + name


def test_size_queries_and_validation(lib):
    assert lib.bl_padded_k(5460) == 5632 and lib.bl_padded_k(4096) == 4096
    assert lib.pack_ternary_bytes(4096, 4096, 0) == 4096 * 4096 // 4
    assert lib.pack_ternary_bytes(17, 100, 0) == 32 * 256 // 4
    assert lib.pack_ternary_bytes(4096, 11008, 1) == 4096 // 4 * 11008
    assert lib.quantize_act_bytes(0, 3, 4096) == 3 * 2048
    assert lib.quantize_act_bytes(1, 3, 5460) == 3 * 5632
    assert lib.quantize_act_bytes(2, 3, 3200) == 3 * 3328 // 2
    assert lib.bitlinear_workspace_bytes(0, 16384, 12288, 4096) >= 16384 * 2048 + 16384 * 4
    # validation happens before any launch: null pointers and bad sizes are rejected on the host
    assert lib.pack_ternary(None, 0, 4, 4, 1e-5, 0, None, None, None, 0, None) == -1
    assert lib.quantize_act(None, 0, 1, 1, 0, 0, 1e-5, None, None, None, None, None) == -1
    assert lib.bitlinear_a4(None, 0, 1, 1, None, 0, None, 1, 1e-5, 0, None, 0, None, None, 0, None) == -1
    assert lib.bitlinear_a4(16, 0, 1, 40000, 16, 0, 16, 1, 1e-5, 0, 16, 0, None, None, 0, None) == -2
    assert lib.bitlinear_a8_sparse(16, 0, 4, 64, 65, 16, 0, 16, 8, 1e-5, 16, 0, None, 16, 1 << 20, None) == -1
    assert lib.bl_status_string(-4).decode().startswith("workspace")


def test_binding_loads_where_torch_has_no_gpu_support(lib):
    """Sizes, constants and signatures need no device: the module loads on a torch without the raw stream call."""
    code = ("import torch; hasattr(torch._C, '_cuda_getCurrentRawStream') and delattr(torch._C, '_cuda_getCurrentRawStream')\n"
            "from paper_2411_04965_amd import binding\n"
            "assert binding.lib().bl_padded_k(5460) == 5632\n")
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
