"""The batched tuner's candidates: only parameters that the form they are swept
in obeys, and the library's defaults among them."""
from paper_2207_00257_amd import tune

CUS = 256
BASE = dict(block=256, unroll=8, map_unroll=4, grid=2048, tile_log2=15, short_regs=4, graph=1, map_block=1024,
            map_grid=1024, keep_mib=256, resident_segments=64, resident_grid=768, wave_max=2048, wave_grid=1024)
OFF = dict(BASE, resident_segments=0)


def _varied(candidates):
    return {k for p in candidates for k, v in p.items() if BASE.get(k) != v}


def test_resident_and_wavefront_candidates_hold_the_defaults():
    resident = list(tune.resident_candidates(BASE, CUS))
    assert _varied(resident) == {"resident_segments", "resident_grid"}
    assert BASE in resident and BASE in tune.resident_candidates(BASE, CUS, quick=True)
    assert all(p["resident_grid"] >= max(1, p["resident_segments"]) for p in resident)
    wave = list(tune.wave_candidates(BASE))
    assert _varied(wave) == {"wave_max"} and BASE in wave


def test_tiles_are_swept_in_the_form_that_has_them():
    # every row resident: nothing of the tiles shows
    for candidates in (tune.tile_candidates(BASE, CUS, 1 << 20), tune.map_candidates(BASE, CUS), tune.keep_candidates(BASE, 1 << 20)):
        assert not list(candidates)
    assert _varied(tune.tile_candidates(BASE, CUS, (1 << 20) + 1)) == {"tile_log2"}
    assert _varied(tune.keep_candidates(BASE, (1 << 20) + 1)) == {"keep_mib"}
    assert _varied(tune.tile_candidates(OFF, CUS, 5)) == {"resident_segments", "block", "unroll", "tile_log2", "short_regs", "grid"}
    assert _varied(tune.map_candidates(OFF, CUS)) == {"resident_segments", "map_block", "map_unroll", "map_grid"}
    assert list(tune.keep_candidates(OFF, 5))


def test_serving_candidates_obey_resident_rows():
    for quick in (False, True):
        space = tune.serve_candidates(CUS, quick)
        assert space and all(set(p) == {"resident_grid", "wave_max", "tile_log2", "graph"} for p in space)
    assert dict(resident_grid=768, wave_max=2048, tile_log2=15, graph=1) in tune.serve_candidates(CUS)
