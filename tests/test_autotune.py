"""The autotuner's bookkeeping, without a GPU: which candidates are timed and which one is picked."""
from paper_2601_09417_amd import trainer


def test_equal_schedules_are_timed_once(monkeypatch):
    """Candidates that differ in the forward's LDS batch only are the same step: one series of steps for them, so that
    the pick does not depend on which of their timings came out lower.  The first series of a process is slower than the
    same one later; it is run again and does not count."""
    series = []

    class Tuner:
        def __init__(self, *args, tile, sort_bits, lds_batch, lds_batch_bwd, **kw):
            self.key = (tile, sort_bits, lds_batch_bwd)

    def time_steps(ft, steps, warmup):
        series.append(ft.key)
        ms = {(16, 8, 0): 2.0, (16, 4, 0): 2.05}.get(ft.key, 3.0)
        return ms * 1.05 if len(series) == 1 else ms

    monkeypatch.setattr(trainer, "FineTuner", Tuner)
    monkeypatch.setattr(trainer, "_time_steps", time_steps)
    r = trainer.autotune(None, [], None)
    schedules = list(dict.fromkeys((t, b, kb) for t, b, k, kb in trainer.TUNE_CANDIDATES))
    assert len(schedules) < len(trainer.TUNE_CANDIDATES)
    assert series == schedules[:1] + schedules
    assert [(d["tile"], d["sort_bits"], d["lds_batch"], d["lds_batch_bwd"]) for d in r["table"]] == \
        list(trainer.TUNE_CANDIDATES)
    assert (r["tile"], r["sort_bits"], r["lds_batch"], r["lds_batch_bwd"], r["ms"]) == (16, 8, 0, 0, 2.0)
