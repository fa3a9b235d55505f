"""The autotuner's cache: a stored choice is applied without timing only to the same basis and to a
library whose present form of the encoder was among the timed ones."""
import json
import types

import pytest

from paper_1806_04374_amd import autotune


class Library:
    """What autotune.tune calls, with the form that "auto" takes and a count of the timings."""

    def __init__(self, form):
        self.form, self.timed, self.launch = form, 0, ("auto", 0)

    def rsc_get_launch(self, h):
        return self.launch

    def rsc_set_launch(self, h, tile, bpc):
        self.launch = (tile, bpc)

    def rsc_encode_info(self, h, K):
        return (self.form if self.launch[0] == "auto" else self.launch[0]), 0.0

    def rsc_autotune_encode(self, h, x, K, reps):
        self.timed += 1
        self.launch = (self.form, 2)
        return [(self.form, 1, 0.5), (self.form, 2, 0.4), ("32", 1, 0.9)]


def _handle(**more):
    return types.SimpleNamespace(N=11, S=5, T=5, B=55, M=64, R=64, prec="fp32", **more)


@pytest.fixture
def tuned(tmp_path, monkeypatch):
    def run(form, handle=None):
        lib = Library(form)
        monkeypatch.setattr(autotune, "rsc", lib)
        out = autotune.tune(handle or _handle(), types.SimpleNamespace(shape=(1000, 55)), 4, path=str(tmp_path / "c.json"))
        return lib, out
    return run


def test_a_stored_choice_is_applied(tuned):
    lib, first = tuned("auto")
    assert lib.timed == 1 and not first["cached"]
    lib, again = tuned("auto")
    assert lib.timed == 0 and again["cached"] and lib.launch == ("auto", 2)


def test_a_choice_without_the_present_form_is_timed_again(tuned):
    """A cache from before the library had its screened form holds the tiles "16" and "32" only."""
    tuned("16")
    lib, out = tuned("auto")
    assert lib.timed == 1 and not out["cached"] and lib.launch == ("auto", 2)
    lib, out = tuned("auto")
    assert lib.timed == 0 and out["cached"]


def test_bases_have_entries_of_their_own(tuned, tmp_path):
    tuned("auto")
    lib, out = tuned("auto", _handle(Ts=[1, 3, 5, 5, 5]))
    assert lib.timed == 1 and not out["cached"]
    assert len(json.loads((tmp_path / "c.json").read_text())) == 2
