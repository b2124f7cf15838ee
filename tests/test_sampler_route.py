"""Which samplers ``run`` may hand to the one-launch form: only those whose loop would make exactly the library's own
calls.  Whoever replaces one of them (a denoiser object of their own, a subclass that changes ``window``, ``sdden_eval``
or a context call, a patched instance) has the loop run, on the CPU here with recording stand-ins for the library."""
import pytest
import torch

from paper_2501_05370_amd import binding, sampler
from paper_2501_05370_amd.sampler import (DiffusionSampler, EfficientFrozenSampler, IndependentDrafterSampler, LangevinSampler,
                                          WindowBuffers)


@pytest.fixture
def calls(monkeypatch):
    """Names of the entry points called, in order; sd_advance ends the run."""
    c = []
    monkeypatch.setattr(binding.Denoiser, "__del__", lambda self: None, raising=False)
    monkeypatch.setattr(binding.Context, "__del__", lambda self: None, raising=False)

    def record(cls, name, result=None):
        def call(self, *a, **k):
            c.append(name)
            if name == "sd_advance":
                a[8].fill_(0)
            return result
        monkeypatch.setattr(cls, name, call)

    for name in ("sd_init_state", "sd_draft", "sd_draft_step", "sd_verify", "sd_advance", "sd_langevin_window",
                 "sd_set_draft_mirror", "sd_set_active_count"):
        record(binding.Context, name)
    record(binding.Context, "sd_langevin_chains", True)
    record(binding.Denoiser, "sdden_eval")
    record(binding.Denoiser, "sdden_set_active_count")
    record(binding.Denoiser, "sdden_run", True)
    monkeypatch.setattr(sampler, "_LOOP_CALLS", sampler._loop_calls())    # the recorders stand for the library's own
    return c


def _make(cls, den_cls=binding.Denoiser, ctx_cls=binding.Context, B=2, d=4, K=3):
    s = cls.__new__(cls)
    s.ctx = ctx_cls.__new__(ctx_cls)
    s.ctx.d, s.ctx.K, s.ctx.T = d, K, 5
    s.buf = b = WindowBuffers(B, d, K, device="cpu")
    s.den, s.draft_den = den_cls.__new__(den_cls), den_cls.__new__(den_cls)
    s.mirror = None
    b.mp, b.Dp, b.cur, b.kcur = torch.zeros(B, K, d), torch.zeros(B, d), [torch.zeros(B, d)] * 2, [torch.zeros(B)] * 2
    b.Dfz, b.X_ext, b.krow_ext, b.Dq_ext = (torch.zeros(B, d), torch.zeros(B, K + 1, d), torch.zeros(B, K + 1, dtype=torch.int32),
                                            torch.zeros(B, K + 1, d))
    s.means, s.logw, s.comp_std, s.gamma, s.M = torch.zeros(2, d), torch.zeros(2), 1.0, 0.1, 2
    return s


DIFFUSION = [DiffusionSampler, EfficientFrozenSampler, IndependentDrafterSampler]
IDS = torch.arange(2)


@pytest.mark.parametrize("cls", DIFFUSION + [LangevinSampler])
def test_the_librarys_own_calls_take_one_launch(cls, calls):
    _make(cls).run(IDS)
    assert ("sd_langevin_chains" if cls is LangevinSampler else "sdden_run") in calls
    assert "sd_advance" not in calls

    class Derived(cls):                                  # a subclass that changes neither loop nor calls
        def note(self):
            return 1
    calls.clear()
    _make(Derived).run(IDS)
    assert "sd_advance" not in calls


class _OwnNetwork:
    """A user's denoiser: has sdden_eval and nothing else of Denoiser."""
    def __init__(self):
        self.evals = 0

    def sdden_eval(self, R, X, krow, out):
        self.evals += 1


@pytest.mark.parametrize("cls", DIFFUSION)
def test_a_denoiser_object_with_sdden_eval_only(cls, calls):
    s = _make(cls)
    s.den, s.draft_den = _OwnNetwork(), _OwnNetwork()
    s.run(IDS)
    assert s.den.evals >= 1 and "sd_advance" in calls
    s = _make(cls)
    if cls is IndependentDrafterSampler:                 # the draft model alone
        s.draft_den = _OwnNetwork()
        s.run(IDS)
        assert s.draft_den.evals == 3 and "sdden_run" not in calls


@pytest.mark.parametrize("cls", DIFFUSION)
def test_a_denoiser_subclass_that_changes_the_prediction(cls, calls):
    seen = []

    class Guided(binding.Denoiser):
        def sdden_eval(self, R, X, krow, out):
            super().sdden_eval(R, X, krow, out)
            seen.append(R)
    _make(cls, den_cls=Guided).run(IDS)
    assert seen and "sdden_run" not in calls
    s = _make(cls)
    s.den.sdden_eval = lambda R, X, krow, out: seen.append(R)        # patched on the object
    seen.clear()
    s.run(IDS)
    assert seen and "sdden_run" not in calls


@pytest.mark.parametrize("cls", DIFFUSION + [LangevinSampler])
@pytest.mark.parametrize("what", ["window", "advance"])
def test_a_sampler_subclass_that_changes_the_loop(cls, what, calls):
    seen = []

    def override(self, B, *a):
        seen.append(B)
        return getattr(cls, what)(self, B, *a)
    _make(type("Derived", (cls,), {what: override})).run(IDS)
    assert seen and "sd_advance" in calls
    s, seen2 = _make(cls), []
    plain = getattr(s, what)
    setattr(s, what, lambda B: (seen2.append(B), plain(B)))          # patched on the object
    s.run(IDS)
    assert seen2


@pytest.mark.parametrize("cls,name", [(DiffusionSampler, "sd_draft"), (DiffusionSampler, "sd_verify"), (DiffusionSampler, "sd_advance"),
                                      (EfficientFrozenSampler, "sd_draft"), (IndependentDrafterSampler, "sd_draft_step"),
                                      (LangevinSampler, "sd_langevin_window"), (LangevinSampler, "sd_advance")])
def test_a_context_that_changes_a_call(cls, name, calls):
    seen = []

    def override(self, *a, **k):
        seen.append(name)
        return getattr(binding.Context, name)(self, *a, **k)
    _make(cls, ctx_cls=type("Traced", (binding.Context,), {name: override})).run(IDS)
    assert seen and "sd_advance" in calls


@pytest.mark.parametrize("cls", [DiffusionSampler, EfficientFrozenSampler])
def test_few_chains_of_long_predictions_take_the_loop(cls, calls):
    """One chain, long windows, thousands of pairs per wavefront: the separate calls; up to 256 coordinates, many chains, or a
    denoiser that does not say how many components it has: one launch."""
    def launches(components, **kw):
        calls.clear()
        s = _make(cls, **kw)
        s.ctx.T = 1000
        if components:
            s.den.components = components
        s.run(torch.arange(kw.get("B", 2)))
        return "sdden_run" in calls
    assert not launches(64, B=1, d=1000, K=16)
    assert not launches(48, B=4, d=300, K=64)
    assert launches(48, B=4, d=200, K=64)                # positions side by side in the one launch
    assert launches(64, B=1, d=256, K=64)
    assert launches(64, B=200, d=1000, K=16)
    assert launches(32, B=1, d=64, K=64)
    assert launches(8, B=1, d=2, K=4)
    assert launches(0, B=1, d=1000, K=16)
    assert launches(65, B=1, d=1000, K=16)               # the library itself says no to these
