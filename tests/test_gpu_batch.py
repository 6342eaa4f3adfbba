"""GPU parity of the batched form (logfx_extract_batch): many uneven tiles in
one launch per pass, persistent or not, replayed from a hipGraph or not.
Every tile is an independent image: its map must equal the single-image
call bit for bit, and the oracle under the band rule."""
import numpy as np
import pytest

from paper_1304_3992_amd import logfx, scenes
from parity import compare, masks, run_oracle, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    c = logfx.Context(0)
    yield c
    c.close()


def _tiles(n=9, seed=31, lo=40, hi=700):
    return scenes.config3(n=n, seed=seed, base_seed=5000 + seed, lo=lo, hi=hi)


def _singles(ctx, devs, params):
    return [ctx.extract(t, params, report=True) for t in devs]


@pytest.mark.parametrize("persistent,graph", [(1, 1), (0, 1), (1, 0), (0, 0)])
def test_batch_equals_single_calls_and_oracle(ctx, persistent, graph):
    import torch
    tiles = _tiles()
    orc_t, lib_t = masks()
    params = logfx.Params(*lib_t)
    devs = [to_device(t) for t in tiles]
    ctx.set_option(logfx.OPT_PERSISTENT, persistent)
    ctx.set_option(logfx.OPT_GRAPH, graph)
    try:
        outs, reps = ctx.extract_batch(devs, params, report=True)
    finally:
        ctx.set_option(logfx.OPT_PERSISTENT, 0)
        ctx.set_option(logfx.OPT_GRAPH, 1)
    torch.cuda.synchronize()
    singles = _singles(ctx, devs, params)
    torch.cuda.synchronize()
    for i, t in enumerate(tiles):
        F = outs[i].cpu().numpy()
        Fs, rs = singles[i]
        assert np.array_equal(F, Fs.cpu().numpy()), i
        assert reps[i] == rs, i
        compare(F, run_oracle(t, orc_t), smooth=True)


def test_graph_replays_match_eager(ctx):
    """The captured graph is replayed several times with eager work and
    synchronisations in between; every replay must equal the eager result,
    including after new input data in the same buffers."""
    import torch
    tiles = _tiles(n=6, seed=32)
    _, lib_t = masks()
    params = logfx.Params(*lib_t)
    devs = [to_device(t) for t in tiles]
    outs = [torch.empty(t.shape, dtype=torch.uint8, device="cuda") for t in tiles]
    ctx.set_option(logfx.OPT_GRAPH, 0)
    eager = [o.clone() for o in ctx.extract_batch(devs, params)]
    ctx.set_option(logfx.OPT_GRAPH, 1)
    for rep in range(4):
        for o in outs:
            o.fill_(7)
        ctx.extract_batch(devs, params, outs)
        torch.cuda.synchronize()
        junk = torch.ones(1 << 20, device="cuda").sum()   # unrelated eager work
        torch.cuda.synchronize()
        for o, e in zip(outs, eager):
            assert torch.equal(o, e), rep
        del junk
    # new pixels in the same buffers: the replay must pick them up
    flipped = [np.ascontiguousarray(t[::-1]) for t in tiles]
    for d, f in zip(devs, flipped):
        d.copy_(to_device(f))
    ctx.extract_batch(devs, params, outs)
    ctx.set_option(logfx.OPT_GRAPH, 0)
    ref = ctx.extract_batch(devs, params)
    ctx.set_option(logfx.OPT_GRAPH, 1)
    torch.cuda.synchronize()
    for o, r in zip(outs, ref):
        assert torch.equal(o, r)


def test_batch_rejects_mixed_dtypes(ctx):
    _, lib_t = masks()
    params = logfx.Params(*lib_t)
    a = to_device(np.zeros((20, 20), np.uint8))
    b = to_device(np.zeros((20, 20), np.uint16))
    with pytest.raises(logfx.LogfxError) as e:
        ctx.extract_batch([a, b], params)
    assert e.value.code == logfx.EINVAL


def test_batch_edge_shapes(ctx):
    """Degenerate members of a batch: a single pixel, one row, one column,
    and a tile narrower than the halo, next to an ordinary tile."""
    import torch
    rng = np.random.default_rng(33)
    tiles = [np.array([[5]], np.uint16), rng.integers(0, 256, (1, 300)).astype(np.uint16),
             rng.integers(0, 256, (300, 1)).astype(np.uint16),
             rng.integers(0, 256, (3, 7)).astype(np.uint16),
             scenes.config3(n=1, seed=34, lo=300, hi=400)[0]]
    orc_t, lib_t = masks()
    params = logfx.Params(*lib_t)
    outs = ctx.extract_batch([to_device(t) for t in tiles], params)
    torch.cuda.synchronize()
    for t, o in zip(tiles, outs):
        compare(o.cpu().numpy(), run_oracle(t, orc_t), smooth=True)


def test_config3_full_batch(ctx):
    """The 64 uneven tiles (sides log-uniform in [256, 4096]) in one call at
    the benchmark's launch configuration, each against the oracle."""
    import torch
    tiles = scenes.config3()
    orc_t, lib_t = masks()
    params = logfx.Params(*lib_t)
    outs, reps = ctx.extract_batch([to_device(t) for t in tiles], params, report=True)
    torch.cuda.synchronize()
    total = 0
    for t, o, r in zip(tiles, outs, reps):
        o_ref = run_oracle(t, orc_t)
        compare(o.cpu().numpy(), o_ref, smooth=True)
        np.testing.assert_allclose(r["sigma_g"], o_ref["stats"][:2], rtol=1e-12)
        total += t.size
    assert total > 50_000_000


def test_autotuner_choice_cache_and_unchanged_output(tmp_path):
    """The tuner picks strip heights among its candidates, keeps the outputs
    bit-identical, writes its cache, and a second context takes the choice
    from the cache without measuring."""
    import torch
    img = scenes.panchromatic(900, 1300, 41, n_rect=150, noise_sigma=4.0)
    _, lib_t = masks()
    params = logfx.Params(*lib_t)
    dev = to_device(img)
    cache = str(tmp_path / "tune.jsonl")
    with logfx.Context(0) as c1:
        ref = c1.extract(dev, params).clone()
        res = c1.tune(dev, params, reps=2, cache=cache)
        assert res["from_cache"] == 0
        assert res["rows1"] in (32, 40, 48, 56, 64, 96) and res["rows2"] in (32, 40, 48, 56, 64, 96)
        assert c1.get_option(logfx.OPT_ROWS1) == res["rows1"]
        assert torch.equal(c1.extract(dev, params), ref)
    with logfx.Context(0) as c2:
        res2 = c2.tune(dev, params, reps=2, cache=cache)
        assert res2["from_cache"] == 1
        assert (res2["rows1"], res2["rows2"]) == (res["rows1"], res["rows2"])
        assert torch.equal(c2.extract(dev, params), ref)
    tiles = _tiles(n=5, seed=42)
    devs = [to_device(t) for t in tiles]
    with logfx.Context(0) as c3:
        refs = [o.clone() for o in c3.extract_batch(devs, params)]
        resb = c3.tune(devs, params, reps=2, cache=cache)
        assert resb["persistent"] in (0, 1)
        outs = c3.extract_batch(devs, params)
        torch.cuda.synchronize()
        for o, r in zip(outs, refs):
            assert torch.equal(o, r)


def test_tune_cache_from_environment(tmp_path, monkeypatch):
    """logfx_tune with no cache path uses the file LOGFX_TUNE_CACHE names:
    the first context measures and writes it, a second one reads it."""
    img = scenes.panchromatic(300, 700, 43, n_rect=40, noise_sigma=4.0)
    _, lib_t = masks()
    params = logfx.Params(*lib_t)
    dev = to_device(img)
    cache = tmp_path / "env_tune.jsonl"
    monkeypatch.setenv("LOGFX_TUNE_CACHE", str(cache))
    with logfx.Context(0) as c1:
        res = c1.tune(dev, params, reps=1)
    assert res["from_cache"] == 0 and cache.exists() and '"key"' in cache.read_text()
    with logfx.Context(0) as c2:
        assert c2.tune(dev, params, reps=1)["from_cache"] == 1


@pytest.mark.parametrize("graph", [1, 0])
def test_alternating_batches_queued_without_sync(ctx, graph):
    """Three different batches (their own tile counts and image tables) and
    repeats of them, queued on one stream with no host synchronization in
    between: each upload goes through the pinned staging set of its turn, an
    unchanged batch uploads nothing, and every output equals the batch's own
    output computed alone."""
    import torch
    _, lib_t = masks()
    params = logfx.Params(*lib_t)
    sets = [_tiles(n=5, seed=61, lo=60, hi=500), _tiles(n=7, seed=62, lo=60, hi=500),
            _tiles(n=3, seed=63, lo=300, hi=900)]
    devs = [[to_device(t) for t in s] for s in sets]
    ctx.set_option(logfx.OPT_GRAPH, graph)
    try:
        refs = []
        for d in devs:
            refs.append([o.clone() for o in ctx.extract_batch(d, params)])
        torch.cuda.synchronize()
        order = [0, 1, 2, 2, 0, 0, 1, 2, 1, 0]
        outs = [[torch.full(t.shape, 7, dtype=torch.uint8, device="cuda") for t in s] for s in sets]
        results = []
        for k in order:
            ctx.extract_batch(devs[k], params, outs[k])
            results.append((k, [o.clone() for o in outs[k]]))
        torch.cuda.synchronize()
        for k, got in results:
            for g, r in zip(got, refs[k]):
                assert torch.equal(g, r), k
    finally:
        ctx.set_option(logfx.OPT_GRAPH, 1)


@pytest.mark.parametrize("field,value,rc", [("width", 0, logfx.EINVAL), ("height", 0, logfx.EINVAL),
                                            ("height", -5, logfx.EINVAL), ("width", 1 << 40, logfx.EINVAL),
                                            ("height", 1 << 62, logfx.EUNSUPPORTED), ("data", None, logfx.EINVAL)])
def test_invalid_images_of_a_gated_batch_are_refused(field, value, rc):
    """Every image is checked before its sizes are used (the gate's cell
    layout divides by them), and the parameters before they are read."""
    import ctypes
    import torch
    from oracle import gate as og
    lib = logfx.load()
    dev = to_device(scenes.panchromatic(130, 140, 3, n_rect=5, noise_sigma=2.0))
    params = logfx.Params(*masks()[1], smooth=logfx.SMOOTH_GATE)
    outs = [torch.empty_like(dev) for _ in range(2)]
    descs = (logfx.logfx_image * 2)(logfx.image(dev), logfx.image(dev))
    ptrs = (ctypes.c_void_p * 2)(*(o.data_ptr() for o in outs))
    with logfx.Context(0) as c:
        c.gate_set_params(og.init(2))

        def call(p):
            return lib.logfx_extract_batch(c.ptr, 2, descs, p, ctypes.cast(ptrs, ctypes.POINTER(ctypes.c_void_p)),
                                           None, None)

        want = [o.clone() for o in c.extract_batch([dev, dev], params)]
        setattr(descs[1], field, value)
        assert call(ctypes.byref(params.c)) == rc
        assert call(None) == logfx.EINVAL
        got = c.extract_batch([dev, dev], params)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))


TUNE_SCRIPT = r"""
import os
import sys
import time
sys.path[:0] = [%r, %r]
import numpy as np
import torch
from paper_1304_3992_amd import logfx, scenes
from parity import masks, to_device
rng = np.random.default_rng(1)
small = to_device(scenes.config1())
large = to_device(rng.integers(0, 256, (8192, 4100)).astype(np.uint8))
deep = to_device(rng.integers(0, 65536, (512, 512)).astype(np.uint16))
params = logfx.Params(*masks()[1])


def call(c, name, d):
    print("CALL", name, file=sys.stderr, flush=True)
    c.extract(d, params)


def us(c, d):
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(200):
            c.extract(d, params)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best * 5e3


with logfx.Context(0) as c:
    for name, d in (("small", small), ("large", large), ("deep", deep)):
        call(c, name, d)
    before = us(c, small)
    c.tune(large, params, reps=2)
    for name, d in (("small", small), ("deep", deep)):
        call(c, name, d)
    c.tune(small, params, reps=20)
    for name, d in (("large", large), ("deep", deep)):
        call(c, name, d)
    print("RATIO", us(c, small) / before)
"""


def test_tuning_one_call_leaves_others_their_heights():
    """Strip heights tuned on a large image are not those of a small one
    (nor the other way round, nor of a call of the other arithmetic), which
    go on choosing by their own size; and a call is no slower tuned than
    untuned (512 x 512: 17 us, 41 with the shortest strips of the list)."""
    import os
    import re
    import subprocess
    import sys
    here = os.path.dirname(os.path.abspath(__file__))
    r = subprocess.run([sys.executable, "-c", TUNE_SCRIPT % (os.path.dirname(here), here)],
                       env=dict(os.environ, LOGFX_LOG="1"), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    rows = {}
    for name, a, b in re.findall(r"CALL (\w+)\n\[liblogfx\] extract: .*?\(rows (\d+)/(\d+)\)", r.stderr):
        rows.setdefault(name, []).append((int(a), int(b)))
    assert len(rows["small"]) == 2 and len(rows["large"]) == 2 and len(rows["deep"]) == 3, rows
    assert all(len(set(v)) == 1 for v in rows.values()), rows
    assert rows["small"][0][0] < 32 and rows["large"][0] == (48, 64), rows
    assert float(re.search(r"RATIO ([\d.]+)", r.stdout).group(1)) < 1.3, r.stdout
