"""What the per-call entry points and the training driver accept and refuse (host code only)."""
import numpy as np
import pytest

from paper_1511_05950_amd import binding, driver


def fast():
    binding.load()
    return binding._fast


@pytest.mark.parametrize("call, args", [
    ("push_gradient", (None, 1.0)),
    ("pull_weights", (None, 0, 2.0)),
    ("pull_weights", (None, 0.0, 2)),
    ("get_minibatch", (None, 1.5, 0, 0)),
    ("push_gradient_external", (None, 0, 3.0)),
    ("calc_gradient", (None, [0, 1.0], None)),
])
def test_integer_arguments_refuse_floats(call, args):
    with pytest.raises(TypeError):
        getattr(fast(), call)(*args)


@pytest.mark.parametrize("call, args", [
    ("push_gradient", (None, np.int64(1))),
    ("pull_weights", (None, np.int32(0), 0)),
    ("calc_gradient", (None, np.array([0, 1]), None)),
])
def test_integer_arguments_take_numpy(call, args):
    with pytest.raises(binding.SasgdError):      # the missing context, not the argument
        getattr(fast(), call)(*args)


class _Context:
    """The calls a training run makes, without a network behind them."""

    def __init__(self, c):
        self.c, self.ts, self.asked = c, 0, []

    def timestamp(self):
        return self.ts

    def getMinibatch(self, learner, x, y):
        pass

    def pullWeights(self, learner, tau):
        assert type(tau) is int
        self.asked.append(tau)
        return self.ts - tau

    def calcGradient(self, learners, loss=None):
        pass

    def pushGradient(self, learner):
        return 0

    def sumGradients(self):
        pass

    def applyUpdate(self):
        self.ts += 1

    def flush(self):
        pass


@pytest.mark.parametrize("form", [np.asarray, lambda s: np.asarray(s, dtype=np.float64), lambda s: s, lambda s: np.asarray(s, dtype=object)])
def test_schedule_forms(form):
    """Arrays of any type, lists, and rows with more entries than a window has gradients give the same run."""
    c, rows = 2, [[0, 0], [1, 0], [0, 1], [2, 1], [1, 0]]
    log = []
    for schedule in (np.asarray(rows), form([r + [7] for r in rows])):
        for run in (driver.run_softsync_batched, driver.run_softsync):
            ctx = _Context(c)
            run(ctx, schedule, lambda i, l: (None, None), 4)
            log.append((run.__name__, ctx.asked))
    assert log[0] == log[2] and log[1] == log[3]


class _AsItGoes:
    """A schedule that is made while the run goes on: length and rows by index only, rows that know nothing but their entries, none
    of them further ahead of the server than the learners can be."""

    def __init__(self, ctx, rows, ahead):
        self.ctx, self.rows, self.ahead = ctx, rows, ahead

    def __len__(self):
        return len(self.rows)

    def __iter__(self):
        raise TypeError("rows are fetched by index")

    def __getitem__(self, k):
        assert k <= self.ctx.ts + self.ahead
        return dict(enumerate(self.rows[k]))


@pytest.mark.parametrize("run, ahead", [(driver.run_softsync, 0), (driver.run_softsync_batched, 2)])
def test_schedule_made_while_the_run_goes_on(run, ahead):
    c, lam, rows = 2, 4, [[0, 0], [1, 0], [0, 1], [2, 1], [1, 0], [0, 0], [3, 2]]
    asked = []
    for schedule in (lambda ctx: _AsItGoes(ctx, rows, ahead), lambda ctx: np.asarray(rows)):
        ctx = _Context(c)
        run(ctx, schedule(ctx), lambda i, l: (None, None), lam)
        asked.append(ctx.asked)
    assert asked[0] == asked[1] and len(asked[0]) == c * len(rows)
