"""The native marshalling (binding/bind.cpp) where no device is needed: what it clears and what it lets through."""
import pytest

from paper_2604_12452_amd import lca


@pytest.fixture
def bind():
    lca.load()
    assert lca._bind is not None, "the native marshalling was not built"
    return lca._bind


def _call(bind, desc, layout=None):
    if layout is not None:
        return bind.decode_attn_cached(desc, layout, *[None] * 8)
    return bind.dense_attn(desc, *[None] * 7)


class _Stop(Exception):
    """What a signal handler might raise."""


@pytest.mark.parametrize("error", [KeyboardInterrupt, _Stop, MemoryError])
@pytest.mark.parametrize("owner,field", [(lca.Desc, "g"), (lca.Desc, "scale"), (lca.CacheLayout, "m_cap")])
def test_an_exception_that_is_not_about_the_arguments_ends_the_call(bind, monkeypatch, error, owner, field):
    desc, layout = lca.Desc(B=1, L=64, H=2, S=1, d_pool=64, d_sel=64, g=4, w=8, mode=lca.MODE_GQA), lca.CacheLayout(20, 20)

    def read(self):
        raise error("from elsewhere")
    monkeypatch.setattr(owner, field, property(read, lambda self, v: None), raising=False)
    with pytest.raises(error):
        _call(bind, desc, layout if owner is lca.CacheLayout else None)


def test_a_missing_field_is_left_to_python(bind):
    desc = lca.Desc(B=1, L=64, H=2, S=1, d_pool=64, d_sel=64, g=4, w=8, mode=lca.MODE_GQA)
    assert _call(bind, desc) == -1                    # (no tensors)
    del desc.g
    assert _call(bind, desc) == -1
    with pytest.raises(AttributeError):
        lca.condense(desc, *[None] * 8)


@pytest.mark.gpu
@pytest.mark.parametrize("error", [KeyboardInterrupt, _Stop])
def test_an_exception_while_the_stream_is_asked_for_ends_the_call(bind, error):
    """A stream whose address raises once: without the exception the call would have gone on the second time."""
    import torch
    desc = lca.Desc(B=1, L=64, H=2, S=1, d_pool=64, d_sel=64, g=4, w=8, mode=lca.MODE_GQA)
    t = [torch.zeros(1, 64, h, 64, dtype=torch.bfloat16, device="cuda") for h in (2, 1, 1, 2)]

    class Stream:
        asked = 0

        @property
        def cuda_stream(self):
            self.asked += 1
            if self.asked == 1:
                raise error("from elsewhere")
            return torch.cuda.current_stream().cuda_stream

    with pytest.raises(error):
        lca.dense_attn(desc, *t, None, lca.alloc_workspace(desc), stream=Stream())


def test_another_torch_is_refused(bind):
    """The module reads tensors by accessors compiled into it: one built for another torch, or Python, must not be used."""
    addresses = dict.fromkeys(lca.EXPORTS, 1)
    for tag in ("torch 2.9.0 abc python 3.10", lca.bind_tag() + " ", ""):
        with pytest.raises(ImportError):
            bind.setup(lca.Desc, lca.CacheLayout, addresses, lca._stream, tag)


@pytest.mark.parametrize("error", [ImportError("built for another"), KeyError("lca_condense"), ValueError("no address")])
def test_a_module_that_does_not_fit_is_done_without(bind, monkeypatch, error):
    import paper_2604_12452_amd as package

    class Other:
        @staticmethod
        def setup(*_):
            raise error
    monkeypatch.setattr(package, "_lcabind", Other, raising=False)
    monkeypatch.setattr(lca, "_bind", None)
    monkeypatch.setitem(__import__("sys").modules, "paper_2604_12452_amd._lcabind", Other)
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        lca._load_bind(lca.load())
    assert lca._bind is None


@pytest.mark.parametrize("error", [ImportError("No module named 'torch'"), FileNotFoundError("g++"), None])
def test_the_library_is_built_without_the_binding(monkeypatch, tmp_path, error):
    """A machine without torch, g++ or their headers: the C library is there, a binding of another build is not."""
    import subprocess

    from paper_2604_12452_amd import build
    lib, bind = tmp_path / "liblca.so", tmp_path / "_lcabind.so"
    bind.write_bytes(b"of another build")

    def fail(force):
        raise error or subprocess.CalledProcessError(1, "g++")
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "BIND", str(bind))
    monkeypatch.setattr(build, "_build_binding", fail)
    with pytest.warns(RuntimeWarning, match="was not built"):
        assert build.build(verbose=False) == str(lib)
    assert lib.exists() and not bind.exists()


def test_a_binding_for_another_torch_is_built_again(monkeypatch, tmp_path):
    from paper_2604_12452_amd import build
    bind = tmp_path / "_lcabind.so"
    monkeypatch.setattr(build, "BIND", str(bind))
    ran = []
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, check: (ran.append(cmd), open(cmd[cmd.index("-o") + 1], "wb").write(lca.bind_tag().encode() + b"\0")))
    bind.write_bytes(b"torch 2.9.0 abc python 3.10\0")
    build._build_binding(False)
    assert len(ran) == 1 and f'-DLCA_BUILT_FOR="{lca.bind_tag()}"' in ran[0]
    build._build_binding(False)
    assert len(ran) == 1
