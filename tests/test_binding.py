"""The checks that stand before the library, in native code: what is refused and how, and what is taken."""
import os
import shutil
import subprocess
import sys

import pytest
import torch


class _Stream:
    cuda_stream = 0


class Wrapped(torch.Tensor):
    """Says of itself that it is on a GPU, without one."""
    @staticmethod
    def __new__(cls, *size, strides=None, device="cuda:0", dtype=torch.float32):
        return torch.Tensor._make_wrapper_subclass(cls, size, strides=strides, device=device, dtype=dtype)

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise NotImplementedError(func)


def rows(n):
    return [Wrapped(3) for _ in range(n)]


class NoIndex:
    def __len__(self):
        return 2

    def __iter__(self):
        return iter(rows(2))


class NoLength:
    def __getitem__(self, i):
        return rows(2)[i]


class Indexed(NoLength):
    def __len__(self):
        return 2


class Short(Indexed):
    def __len__(self):
        return 3


@pytest.fixture
def eng():
    """A handle without a device behind it: the checks come first."""
    from paper_2306_06528_amd import svgd
    e = svgd.Svgd.__new__(svgd.Svgd)
    e._h, e._device = svgd._H(), 0
    return e


@pytest.mark.parametrize("X", [1, None, [[1.0]], torch.zeros(2, 3), torch.zeros(2, 3, device="meta")])
def test_what_is_no_matrix_on_the_gpu(eng, X):
    G = torch.zeros(2, 3)
    for call in (lambda: eng.step(X, G, 0.1, stream=_Stream), lambda: eng.phi(X, G, G, stream=_Stream)):
        with pytest.raises(TypeError, match="X must be a 2-D float32 CUDA tensor"):
            call()


@pytest.mark.parametrize("rows,error", [(([], []), ValueError), (([1], [2]), TypeError), ((3, 4), TypeError),
                                        (([torch.zeros(3)], []), ValueError), (([torch.zeros(3)], [torch.zeros(3)]), TypeError)])
def test_what_is_no_sequence_of_rows(eng, rows, error):
    with pytest.raises(error):
        eng.step_rows(*rows, 0.1, stream=_Stream)


class _Yields:
    """Yields a row, by code of its own."""
    def __iter__(self):
        return iter([torch.zeros(3)])


@pytest.mark.parametrize("second", [torch.zeros(2, 3), _Yields(), [torch.zeros(3)], None])
def test_first_argument_is_refused_before_the_second_is_looked_at(eng, second):
    with pytest.raises(TypeError):
        eng.step_rows(3, second, 0.1, stream=_Stream)


@pytest.mark.skipif(torch.cuda.is_available(), reason="of a machine without a GPU")
def test_what_is_no_matrix_is_named_also_without_a_gpu(eng):
    """The stream and the current device are asked for behind the checks."""
    from paper_2306_06528_amd import svgd
    X, row = torch.zeros(2, 3), [torch.zeros(3)]
    for call in (lambda: eng.step(X, X, 0.1), lambda: eng.phi(X, X, X), lambda: eng.step_rows(row, row, 0.1), lambda: svgd.step_static(X, X, 0.1)):
        with pytest.raises(TypeError, match="float32 CUDA tensor"):
            call()


class Number:
    """An eps, or a stream, that runs `code` when it is asked for."""
    def __init__(self, code):
        self.code = code

    def __float__(self):
        self.code()
        return 0.1

    @property
    def cuda_stream(self):
        self.code()
        return 0


def test_eps_and_stream_are_asked_for_behind_the_checks(eng):
    """And a list of rows that they empty is none of the call's any more."""
    from paper_2306_06528_amd import svgd
    asked = []
    ask = Number(lambda: asked.append(1))
    bad, X = Wrapped(2, 3, dtype=torch.float64), Wrapped(2, 3)
    for call in (lambda: eng.step(X, bad, ask, stream=ask), lambda: eng.phi(X, X, bad, stream=ask), lambda: eng.step_rows([bad], [bad], ask, stream=ask),
                 lambda: svgd.step_static(X, bad, ask, stream=ask)):
        with pytest.raises(TypeError):
            call()
    assert not asked
    X_rows, G_rows = rows(2), rows(2)
    def empty():
        asked.append(1)
        X_rows.clear()
        G_rows.clear()
    with pytest.raises(svgd.SvgdError, match="HANDLE"):
        eng.step_rows(X_rows, G_rows, Number(empty), stream=Number(empty))
    assert len(asked) == 2
    for eps, error in ((None, TypeError), ("x", ValueError), ([1.0], TypeError)):
        with pytest.raises(error):
            eng.step(X, X, eps, stream=_Stream)
        with pytest.raises(error):
            eng.step_rows(rows(2), rows(2), eps, stream=_Stream)


def _outcome(call):
    from paper_2306_06528_amd import svgd
    try:
        call()
    except svgd.SvgdError:
        return "taken"  # by the library, which refuses the handle that is none
    except (TypeError, ValueError) as e:
        return type(e), str(e)
    return "taken"


@pytest.mark.parametrize("X", [
    Wrapped(2, 3), Wrapped(1, 3), Wrapped(2, 1), Wrapped(1, 1), Wrapped(0, 3), Wrapped(2, 0), Wrapped(0, 0), Wrapped(6), Wrapped(2, 3, 1), Wrapped(),
    Wrapped(2, 3, strides=(5, 1)), Wrapped(2, 3, strides=(2, 1)), Wrapped(2, 3, strides=(0, 1)), Wrapped(2, 3, strides=(1, 2)), Wrapped(2, 3, strides=(6, 2)),
    Wrapped(1, 3, strides=(7, 1)), Wrapped(1, 3, strides=(1, 1)), Wrapped(1, 3, strides=(3, 2)), Wrapped(2, 1, strides=(3, 2)), Wrapped(2, 1, strides=(1, 9)),
    Wrapped(2, 1, strides=(0, 1)), Wrapped(1, 1, strides=(0, 0)), Wrapped(0, 3, strides=(1, 1)),
    Wrapped(2, 3, dtype=torch.float64), Wrapped(2, 3, dtype=torch.bfloat16), Wrapped(2, 3, device="cuda:1"), Wrapped(2, 3, device="cpu"),
    Wrapped(1, 3, device="cuda:1"), torch.zeros(2, 3), None, [[1.0]]], ids=lambda X: f"{tuple(X.shape)}{X.stride()}{X.dtype}{X.device}" if torch.is_tensor(X) else str(X))
def test_native_checks_are_those_of_the_calls_that_check_in_python(eng, X):
    """svgd_bandwidth's matrix is checked in Python (svgd._rows_of), those of step, phi and step_static in native code."""
    from paper_2306_06528_amd import svgd
    want = _outcome(lambda: eng._rows(X, "X"))
    assert _outcome(lambda: eng.step(X, X, 0.1, stream=_Stream)) == want
    assert _outcome(lambda: eng.phi(X, X, X, stream=_Stream)) == want
    G = Wrapped(2, 3)
    for x in (X, G):
        def check():
            shape = svgd._rows_of(x, "X")
            if svgd._rows_of(X, "G") != shape:
                raise ValueError("G must have the shape and row stride of X")
            raise TypeError("eps")
        class Eps:
            def __float__(self):
                raise TypeError("eps")
        if not torch.cuda.is_available():  # (without one, nothing is known of the current device)
            svgd_device, svgd._cuda_getDevice = svgd._cuda_getDevice, lambda: x.get_device()
            try:
                assert _outcome(lambda: svgd.step_static(x, X, Eps(), stream=_Stream)) == _outcome(check)
            finally:
                svgd._cuda_getDevice = svgd_device


@pytest.mark.parametrize("binding", ["missing", "untagged", "of_another_torch"])
def test_a_binding_that_does_not_fit_names_the_build(tmp_path, binding):
    from paper_2306_06528_amd import _binding, svgd
    package = tmp_path / "paper_2306_06528_amd"
    package.mkdir()
    here = os.path.dirname(svgd.__file__)
    for name in ("__init__.py", "svgd.py", "libsvgd.so"):
        shutil.copy(os.path.join(here, name), package)
    assert ".cpython-" in os.path.basename(_binding.__file__)  # no other interpreter takes it for its own
    if binding == "untagged":
        (package / "_binding.so").write_bytes(b"")
    if binding == "of_another_torch":
        (package / "_binding.py").write_text("torch_version = '0.0'\n")
    got = subprocess.run([sys.executable, "-c", "import paper_2306_06528_amd.svgd"], cwd=tmp_path, capture_output=True, text=True, timeout=300)
    assert got.returncode and "ImportError" in got.stderr and "paper_2306_06528_amd.build" in got.stderr.splitlines()[-1]


class Sizeless(Wrapped):
    """Asked for its size, it raises an error of its own."""
    @staticmethod
    def __new__(cls, *size):
        return torch.Tensor._make_wrapper_subclass(cls, size, device="cuda:0", dtype=torch.float32, dispatch_sizes_strides_policy="sizes")

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise KeyError("no size")


def test_errors_of_a_tensor_are_raised_as_they_are(eng):
    from paper_2306_06528_amd import svgd
    for call in (lambda: eng.step(Sizeless(2, 3), Wrapped(2, 3), 0.1, stream=_Stream), lambda: eng.phi(Wrapped(2, 3), Sizeless(2, 3), None, stream=_Stream),
                 lambda: eng.step_rows([Sizeless(3)], rows(1), 0.1, stream=_Stream), lambda: svgd.step_static(Sizeless(2, 3), None, 0.1, stream=_Stream)):
        with pytest.raises(KeyError, match="no size"):
            call()


@pytest.mark.parametrize("make", [lambda: set(rows(2)), lambda: (r for r in rows(2)), lambda: dict(enumerate(rows(2))).values(),
                                  lambda: dict(enumerate(rows(2))), lambda: iter(rows(2)), NoIndex, NoLength, lambda: torch.tensor(1.0)])
def test_particles_without_length_or_order_are_refused(eng, make):
    """Also where there are as many scores, of whatever kind."""
    for scores in (rows(2), make()):
        with pytest.raises(TypeError):
            eng.step_rows(make(), scores, 0.1, stream=_Stream)


@pytest.mark.parametrize("make", [lambda: (r for r in rows(2)), lambda: iter(rows(2)), NoLength, lambda: torch.tensor(1.0), lambda: 5])
def test_scores_without_a_length_are_refused(eng, make):
    with pytest.raises(TypeError):
        eng.step_rows(rows(2), make(), 0.1, stream=_Stream)


@pytest.mark.parametrize("make", [list, tuple, lambda r: Indexed()])
def test_sequences_reach_the_library(eng, make):
    """All checks passed: the library is called, and refuses the handle that is none."""
    from paper_2306_06528_amd import svgd
    with pytest.raises(svgd.SvgdError, match="HANDLE"):
        eng.step_rows(make(rows(2)), make(rows(2)), 0.1, stream=_Stream)


def test_sequences_that_yield_fewer_than_they_say(eng):
    for X, G in ((Short(), rows(3)), (rows(3), Short())):
        with pytest.raises((ValueError, IndexError)):
            eng.step_rows(X, G, 0.1, stream=_Stream)


@pytest.mark.gpu
def test_what_is_refused_on_the_gpu():
    from paper_2306_06528_amd import svgd
    n, D = 5, 100
    X, G = torch.randn(n, D, device="cuda"), torch.randn(n, D, device="cuda")
    with svgd.Svgd(n, D) as eng:
        for bad, error in ((X.double(), TypeError), (X[0], TypeError), (X.t(), TypeError), (X.cpu(), TypeError), (X[:, ::2], TypeError),
                           (X[:4], ValueError), (X[:, :99], ValueError), (X[:1].expand(n, D), TypeError), (X.to_sparse(), (TypeError, RuntimeError))):
            for call in (lambda: eng.step(X, bad, 0.1), lambda: eng.phi(X, G, bad), lambda: svgd.step_static(X, bad, 0.1)):
                with pytest.raises(error):
                    call()
        for bad in (None, "x", [1.0]):
            with pytest.raises((TypeError, ValueError)):
                eng.step(X, G, bad)
        with pytest.raises(svgd.SvgdError):
            eng.step(X, G, float("inf"))
        with pytest.raises(svgd.SvgdError):
            eng.step(X, X, 0.1)
        rows = list(X)
        for bad in (rows[:4] + [X[0].double()], rows[:4] + [X[0, :99]], rows[:4] + [X[:, 0]], rows[:4] + [X], rows[:4] + [None]):
            with pytest.raises(TypeError):
                eng.step_rows(rows, bad, 0.1)
            with pytest.raises((TypeError, AttributeError)):
                eng.step_rows(bad[::-1], rows, 0.1)
        with pytest.raises(ValueError):
            eng.step_rows(rows, rows[:4], 0.1)
    with pytest.raises(svgd.SvgdError):
        eng.step(X, G, 0.1)  # closed
    with pytest.raises(svgd.SvgdError):
        eng.step_rows(list(X), list(G), 0.1)


@pytest.mark.gpu
def test_what_is_taken():
    """Views, parameters, numbers that are no floats, tuples and tensors as sequences: the same step."""
    from paper_2306_06528_amd import svgd
    n, D = 6, 333
    g = torch.Generator(device="cuda").manual_seed(0)
    X0, G = torch.randn(n, D, device="cuda", generator=g), torch.randn(n, D, device="cuda", generator=g)
    with svgd.Svgd(n, D) as eng:
        want = X0.clone()
        eng.step(want, G, 0.25)
        for eps in ("0.25", torch.tensor(0.25), torch.tensor(0.25, device="cuda")):
            X = torch.nn.Parameter(X0.clone())
            eng.step(X, torch.nn.Parameter(G), eps)
            assert torch.equal(X.detach(), want)
        for wrap in (list, tuple, lambda M: M):
            X = X0.clone()
            eng.step_rows(wrap(X), wrap(G), 0.25)
            assert float((X - want).abs().max()) <= 1e-6
        one, g1 = X0[:1].clone(), G[:1]
        eng.step(one.as_strided((1, D), (7, 1)), g1, 1)  # a single row: any row stride
        assert torch.equal(one, X0[:1] + g1)
        col, gc = torch.randn(n, 3, device="cuda")[:, :1], torch.randn(n, 3, device="cuda")[:, :1]
        eng.step(col, gc, 0.25)  # a single column
        assert bool(torch.isfinite(col).all())


def test_a_failed_build_names_the_compiler():
    from paper_2306_06528_amd import build
    with pytest.raises(RuntimeError, match=r"^g\+\+ failed"):
        build._run(["g++", "-c", os.path.join(os.path.dirname(__file__), "no_such_file.cpp")])
