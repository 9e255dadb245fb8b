"""Host-side checks of the build script (no GPU)."""
from paper_2007_13055_amd import build


REMARKS = """\
a.hip:10:1: remark: Function Name: kernel_ok [-Rpass-analysis=kernel-resource-usage]
a.hip:10:1: remark:     VGPRs: 64 [-Rpass-analysis=kernel-resource-usage]
a.hip:10:1: remark:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:10:1: remark:     SGPRs Spill: 12 [-Rpass-analysis=kernel-resource-usage]
a.hip:10:1: remark:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]
a.hip:20:1: remark: Function Name: kernel_spills [-Rpass-analysis=kernel-resource-usage]
a.hip:20:1: remark:     ScratchSize [bytes/lane]: 188 [-Rpass-analysis=kernel-resource-usage]
a.hip:20:1: remark:     VGPRs Spill: 70 [-Rpass-analysis=kernel-resource-usage]
"""


def test_spill_detector_names_only_the_spilling_kernel():
    assert build._spilling_kernels(REMARKS) == ["kernel_spills"]
    assert build._spilling_kernels("") == []


def test_kernels_with_hand_placed_loads_are_checked():
    names = [s.rsplit("/", 1)[-1] for s in build.sources()]
    for f in build.NO_SPILL:
        assert f in names


def test_binding_follows_the_header(monkeypatch, tmp_path):
    """An incremental build compiles the native module again when the header that declares the entry points is newer."""
    import os
    from paper_2007_13055_amd import build
    module = tmp_path / "_binding.so"
    module.write_bytes(b"")
    monkeypatch.setattr(build, "BINDING", str(module))
    header = os.path.join(build.ROOT, "include", "bsr_spmm.h")
    newest = max(os.path.getmtime(header), os.path.getmtime(build.BINDING_SRC))
    ran = []
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: ran.append(cmd) or type("R", (), {"returncode": 0})())
    os.utime(module, (newest, newest))
    build.build_binding(force=False)
    assert not ran
    monkeypatch.setattr(build, "BINDING_SRC", str(tmp_path / "source.cpp"))
    (tmp_path / "source.cpp").write_text("")
    os.utime(tmp_path / "source.cpp", (1, 1))
    os.utime(module, (os.path.getmtime(header) - 1,) * 2)             # older than the header alone
    build.build_binding(force=False)
    assert len(ran) == 1
