"""The hash that names a built library: the load check, the autotuner's cache key and the
stored profiles go by it.  It follows the sources and the compiler's flags."""
import pytest

from paper_2006_14927_amd import build, ckv


def test_hash_follows_the_flags(monkeypatch):
    base = build.source_hash()
    assert build.source_hash(["-DX=1"]) != base
    with monkeypatch.context() as m:
        m.setitem(build.FILE_FLAGS, "ckv_kernels.hip", ())
        assert build.source_hash() != base
    with monkeypatch.context() as m:
        m.setattr(build, "COMMON_FLAGS", ("-O2", *build.COMMON_FLAGS[1:]))
        assert build.source_hash() != base
    assert build.source_hash() == base


def test_library_of_other_flags_is_not_taken_for_current(monkeypatch, tmp_path):
    """A library linked with extra flags is loaded as what it is; one of other file flags
    or sources is refused."""
    lib, stamp = tmp_path / "libckv.so", tmp_path / "libckv.sources"
    lib.write_bytes(b"")
    monkeypatch.setattr(ckv, "LIB_PATH", str(lib))
    monkeypatch.setattr(ckv, "_lib", None)
    monkeypatch.setattr(build, "STAMP_PATH", str(stamp))
    stamp.write_text(build.source_hash(["-DX=1"]) + "\n-DX=1\n")
    assert build.built_hash() == build.wanted_hash() != build.source_hash()
    stamp.write_text(build.source_hash() + "\n")
    assert build.built_hash() == build.wanted_hash()
    monkeypatch.setitem(build.FILE_FLAGS, "ckv_kernels.hip", ())
    with pytest.raises(ckv.CkvError, match="other sources or flags"):
        ckv.lib()
