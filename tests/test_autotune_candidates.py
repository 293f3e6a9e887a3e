"""The launches that the render tuner times: whole tiles among them, with the
parameters that give the same launch when they are used later."""
from paper_2504_04564_amd import autotune, vdbc


class _Renderer:
    made = []

    def __init__(self, field, camera, medium, params, mode, background=None):
        self.made.append(dict(params))
        self.launch = lambda: None


def _tuned(monkeypatch, spp, space=None):
    monkeypatch.setattr(_Renderer, "made", [])
    monkeypatch.setattr(vdbc, "Renderer", _Renderer)
    monkeypatch.setattr(autotune, "_median_ms", lambda fn, reps: 1.0)
    _, rows = autotune.tune_render(object(), {}, {}, dict(spp=spp), space=space)
    return _Renderer.made, rows


def test_whole_tiles_and_the_library_choice_are_both_timed(monkeypatch):
    for spp, sizes in ((16, {0, 4, 8, 16}), (6, {0, 4, 6}), (1, {0, 1})):
        made, rows = _tuned(monkeypatch, spp)
        # Renderer takes chunk_spp 0 as the library's choice, spp as whole tiles
        assert {p["chunk_spp"] for p in made} == {r["chunk_spp"] for r in rows} == sizes
        first = [p for p in made if not p["flags"] & vdbc.RENDER_COST_ORDER]
        assert len(first) == len({tuple(sorted(p.items())) for p in first})
        assert len(rows) == len(made) == len(first) + autotune.ORDER_STAGE
    made, _ = _tuned(monkeypatch, 16, dict(chunk_spp=(0,)))
    assert {p["chunk_spp"] for p in made} == {0, 16}
    made, _ = _tuned(monkeypatch, 16, dict(chunk_spp=(8, 32)))
    assert {p["chunk_spp"] for p in made} == {8}
