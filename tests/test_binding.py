"""What the binding of the hot calls refuses before anything reaches a device (tensors in host memory serve for that)."""
import pytest
import torch

from paper_2111_06483_amd import sar


@pytest.fixture(scope="module", autouse=True)
def built():
    sar.native()


def freed():
    import ctypes
    b = sar.Blocks.__new__(sar.Blocks)
    b._h, b._addr, b.flags = None, None, 0
    return b


def test_shapes_and_types_that_must_match():
    h = torch.zeros(4, 8)
    for other in (torch.zeros(8, 4), torch.zeros(4, 8, dtype=torch.bfloat16)):
        with pytest.raises(sar.SarError) as e:
            sar.sar_act_bwd(h, other, sar.SAR_ACT_RELU, torch.zeros(4, 8))
        assert e.value.code == sar.SAR_ERR_INVALID_ARG and "must match" in str(e.value)
        assert "(4, 8) torch.float32" in str(e.value) and str(other.dtype) in str(e.value)


def test_types_the_library_has_not():
    z = torch.zeros(4, 2, 8, dtype=torch.float16)
    with pytest.raises(sar.SarError) as e:
        sar.sar_gat_scores(z, torch.zeros(2, 8), torch.zeros(4, 2))
    assert e.value.code == sar.SAR_ERR_UNSUPPORTED and "torch.float16" in str(e.value)


def test_tensors_that_are_no_plain_memory():
    with pytest.raises(AssertionError, match="contiguous"):
        sar.sar_gat_scores(torch.zeros(2, 8, 4).transpose(1, 2), torch.zeros(4, 8), torch.zeros(2, 4))
    with pytest.raises(TypeError):
        sar.sar_gat_scores([1.0], torch.zeros(2, 8), torch.zeros(4, 2))
    with pytest.raises(ValueError):
        sar.sar_gat_fwd_begin(torch.zeros(4, 2), torch.zeros(4, 2), torch.zeros(4, 16))
    with pytest.raises(TypeError):
        sar.sar_act_bwd(torch.zeros(4), torch.zeros(4), None, torch.zeros(4))


def test_none_for_a_tensor_that_a_call_needs():
    z, a, v = torch.zeros(4, 2, 8), torch.zeros(2, 8), torch.zeros(4, 2)
    for call in (lambda: sar.sar_gat_scores(None, a, v), lambda: sar.sar_gat_scores(z, None, v),
                 lambda: sar.sar_gat_fwd_begin(v, v, None), lambda: sar.sar_gat_fwd_end(v, v, z, None, v),
                 lambda: sar.sar_gat_bwd_begin(None, z, v, v, torch.zeros(4, 2, 4), v),
                 lambda: sar.sar_gat_bwd_end(z, v, a, None, None, a, None),       # (scratch, which the call cannot do without)
                 lambda: sar.sar_gat_bwd_end(None, v, a, None, None, a, v), lambda: sar.sar_error_add(None, None, False, None),
                 lambda: sar.sar_linear_fwd(None, a, v), lambda: sar.sar_linear_fwd(v, None, v),
                 lambda: sar.sar_linear_bwd(v, None, a, None, None, None),
                 lambda: sar.sar_act_bwd(None, v, sar.SAR_ACT_RELU, v)):
        with pytest.raises(AttributeError):
            call()


def test_a_freed_handle():
    for call in (lambda b: sar.sar_spmm_all(b, [], True, torch.zeros(4, 8)),
                 lambda b: sar.sar_spmm_bwd_all(b, torch.zeros(4, 8), True, []),
                 lambda b: sar.sar_gat_fwd_all(b, [], torch.zeros(4, 1), None, torch.zeros(1, 8), 0.2, torch.zeros(4, 1, 8),
                                               torch.zeros(4, 1))):
        with pytest.raises(sar.SarError) as e:
            call(freed())
        assert e.value.code == sar.SAR_ERR_STATE and "freed" in str(e.value)


def test_errors_of_the_library_come_through():
    with pytest.raises(sar.SarError) as e:      # a head wider than a wavefront
        sar.sar_gat_fwd_end(torch.zeros(4, 1), torch.zeros(4, 1), torch.zeros(4, 1, 512), torch.zeros(4, 1, 512),
                            torch.zeros(4, 1))
    assert e.value.code == sar.SAR_ERR_UNSUPPORTED and "64 lanes" in str(e.value)


def test_nothing_to_do_with_no_row():
    sar.sar_linear_fwd(torch.zeros(0, 4), torch.zeros(4, 8), torch.zeros(0, 8))
    sar.sar_gat_scores(torch.zeros(0, 2, 8), a=torch.zeros(2, 8), score=torch.zeros(0, 2))


@pytest.mark.gpu
def test_lists_of_blocks():
    """One tensor per block: missing, of another type, another width, another height, on the host."""
    part = torch.tensor([0, 1, 0, 1], dtype=torch.int32, device="cuda")
    src, dst = torch.tensor([0, 1, 3], device="cuda"), torch.tensor([2, 0, 0], device="cuda")
    b = sar.sar_blocks_build(src, dst, part, 2, 0)
    out, f32 = torch.zeros(2, 8, device="cuda"), dict(device="cuda")
    good = [torch.ones(2, 8, **f32), torch.ones(2, 8, **f32)]
    sar.sar_spmm_all(b, tuple(good), False, out=out)
    assert out.sum().item() == 24.0
    for bad, text in ((torch.ones(2, 8, dtype=torch.bfloat16, **f32), "torch.bfloat16"), (torch.ones(2, 4, **f32), "4 values"),
                      (torch.ones(3, 8, **f32), "2 sources"), (torch.ones(2, 8), "device tensor"),
                      (torch.ones(8, 2, **f32).t(), "contiguous")):
        with pytest.raises(sar.SarError, match=text):
            sar.sar_spmm_all(b, [good[0], bad], False, out)
    with pytest.raises(IndexError):
        sar.sar_spmm_all(b, good[:1], False, out)
    b.close()


@pytest.mark.gpu
def test_lists_of_blocks_are_by_position():
    part = torch.tensor([0, 1, 0, 1], dtype=torch.int32, device="cuda")
    b = sar.sar_blocks_build(torch.tensor([0, 1, 3], device="cuda"), torch.tensor([2, 0, 0], device="cuda"), part, 2, 0)
    out, Z = torch.zeros(2, 8, device="cuda"), torch.ones(2, 2, 8, device="cuda")
    for good in (list(Z), tuple(Z), Z):                  # (one tensor of all blocks' rows is its own list)
        out.zero_()
        sar.sar_spmm_all(b, good, False, out)
        assert out.sum().item() == 24.0
    for bad in (set(Z), iter(Z), (z for z in Z), None, 3):
        with pytest.raises(TypeError):
            sar.sar_spmm_all(b, bad, False, out)
    b.close()


def in_a_copy(tmp_path, name, code):
    """Runs `code` in a fresh interpreter where a copy of the built package is importable as `name` and nothing else of it is."""
    import os
    import shutil
    import subprocess
    import sys
    home = tmp_path / name
    home.mkdir()
    for f in os.listdir(os.path.dirname(sar.__file__)):
        if f.endswith((".py", ".so")):
            shutil.copy(os.path.join(os.path.dirname(sar.__file__), f), home / f)
    return subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True,
                          env={k: v for k, v in os.environ.items() if k != "PYTHONPATH"})


def test_errors_are_of_the_package_the_binding_belongs_to(tmp_path):
    r = in_a_copy(tmp_path, "under_another_name", """
import torch
from under_another_name import sar
try:
    sar.sar_act_bwd(torch.zeros(4, 8), torch.zeros(8, 4), 0, torch.zeros(4, 8))
except sar.SarError as e:
    assert e.code == sar.SAR_ERR_INVALID_ARG and "must match" in str(e), e
else:
    raise AssertionError("not refused")
import sys
assert "paper_2111_06483_amd" not in sys.modules
""")
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("changed", ["torch.__version__ = '2.11.0'", "torch.version.git_version = '0' * 40",
                                     "sys.version_info = (3, 99) + sys.version_info[2:]"])
def test_a_binding_built_for_another_torch_or_interpreter(changed):
    import os
    import subprocess
    import sys
    r = subprocess.run([sys.executable, "-c", """
import sys, torch
from paper_2111_06483_amd import sar
%s
try:
    sar.sar_gat_scores(torch.zeros(0, 2, 8), torch.zeros(2, 8), torch.zeros(0, 2))
except RuntimeError as e:
    assert "_binding.so" in str(e) and "build" in str(e), e
else:
    raise AssertionError("taken")
""" % changed], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_the_libraries_are_built_where_the_binding_cannot_be(tmp_path, monkeypatch):
    import subprocess
    from paper_2111_06483_amd import build

    def no_torch():
        raise ImportError("No module named 'torch'")

    def compiler(cmd, **kwargs):
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build, "HERE", str(tmp_path))
    for name in ("LIB", "BENCH_LIB", "BINDING"):
        monkeypatch.setattr(build, name, str(tmp_path / name))
    monkeypatch.setattr(build, "binding_flags", no_torch)
    monkeypatch.setattr(build.subprocess, "run", compiler)
    with pytest.raises(ImportError):
        build.build()
    assert (tmp_path / "LIB").exists() and (tmp_path / "BENCH_LIB").exists() and not (tmp_path / "BINDING").exists()
