"""The schedules that the selector's classes run, call by call."""

from paper_1203_2946_amd import cmrs, selector


def test_class_runner_takes_the_library_choice_for_strip_groups(monkeypatch):
    """"group" is the product a caller gets by default (the automatic choice of
    stream loads), not one of its two kinds."""
    seen = []
    monkeypatch.setattr(cmrs, "spmv", lambda A, x, out, variant: seen.append((A, variant)))
    monkeypatch.setattr(cmrs, "spmv_colblock", lambda A, plan, x, out, schedule, workspace: seen.append((A, schedule)))
    r = selector.ClassRunner.__new__(selector.ClassRunner)
    r.x = r.y = None
    r.mats, r.plans, r.ws = ({h: h for h in selector.HEIGHTS} for _ in range(3))
    for c in range(selector.N_CLASSES):
        r.run(c)
    want = {"wave": "lds", "wave_nt": "lds_nt", "group": "auto", "colblock4": "concurrent"}
    assert seen == [(h, want[s]) for h, s in selector.CLASSES]
