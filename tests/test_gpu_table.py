"""The fused pipeline's predictor table and decision kernel against the staged
pipeline, which runs the predictor on every candidate: the same bits, at the
sizes where the table, its row map or the decision kernel's forms could go
wrong.  (The staged pipeline itself is checked against the oracle.)"""
import numpy as np
import pytest

from paper_2608_14575_amd import hwr
from paper_2608_14575_amd import synth as S

import gpu_util as G

pytestmark = pytest.mark.gpu


def _feature_bits(lengths):
    return S.f32_to_bf16_bits((np.log(np.asarray(lengths, np.float64)) * 0.125).astype(np.float32))


def _rows():
    """Values of the query feature over every int32 length: each length up to
    256, every bit pattern from there to the largest length's."""
    low = np.unique(_feature_bits(np.arange(1, 257)))
    return low.size + int(_feature_bits([2**31 - 1])[0]) - int(low[-1])


def _lengths(n, seed):
    """Every short length, both sides of each feature step, the largest ones."""
    b = np.arange(int(_feature_bits([2])[0]), int(_feature_bits([2**31 - 1])[0]) + 1, dtype=np.uint32)
    mid = ((b << 16) + 0x8000).astype(np.uint32).view(np.float32).astype(np.float64)      # rounding boundaries
    edge = np.floor(np.exp(8.0 * mid))
    edge = np.concatenate([edge, edge + 1])
    pool = np.concatenate([np.arange(1, 301), edge[(edge >= 1) & (edge < 2**31)], [2**31 - 1, 2**31 - 2]]).astype(np.int64)
    r = np.random.default_rng(seed)
    out = np.concatenate([r.permutation(pool), r.integers(1, 2**31, max(0, n - pool.size))])[:n]
    return out.astype(np.int32)


def _same(a, b):
    for k in a:
        assert a[k].tobytes() == b[k].tobytes(), k


def _both(sp, seed, n, edit=None, candidates=True, **kw):
    pb, st, qs = S.make_problem(sp, seed), S.make_state(sp, seed), S.make_queries(sp, seed, n=n)
    qs.input_len[:] = _lengths(n, seed)
    if edit:
        edit(qs)
    got = []
    for pipeline in ("fused", "staged"):
        r = G.make_router(pb, pipeline=pipeline, **kw)
        r.update(st)
        got.append(G.route_device(r, qs, "bf16", candidates=candidates))
        r.close()
    _same(*got)
    return got[0]


@pytest.mark.parametrize("delta", [-1, 0, 1])
@pytest.mark.parametrize("models,gpus", [(1, 1), (3, 3), (16, 2)])
def test_rows_by_query_and_by_value(models, gpus, delta):
    """Around the batch size where the table changes from one row per query to
    one per feature value; one pair, an odd number, two lane steps."""
    sp = S.spec("C2", n_models=models, n_gpu_types=gpus, hidden=64, embed_dim=64)
    _both(sp, 5, _rows() + delta)


@pytest.mark.parametrize("hidden,heads,kw", [
    (64, 3, {}), (128, 2, dict(cost_weights=[0.0, 0.3, 1.0, 2.0, 0.5, 0.1, 4.0, 0.7])),
    (256, 3, dict(cost_weights=[0.2, 0.9], score_mode=1, **S.PAPER_SLO)), (256, 2, dict(score_mode=1, **S.PAPER_SLO)),
])
def test_every_feature_value(hidden, heads, kw):
    """Both sides of every feature step (1,300 lengths): each query finds the
    row of its own value, at each width, head count and rule."""
    sp = S.spec("C2", hidden=hidden, n_heads=heads, n_models=5, n_gpu_types=3)
    if "score_mode" in kw:
        kw = dict(kw, cost_weight=0.3)
    _both(sp, 6, 1500, **kw)


@pytest.mark.parametrize("embed_dim", [64, 320, 512])
@pytest.mark.parametrize("extra", [-1, 0, 37])
def test_quality_inside_the_decision_kernel(embed_dim, extra):
    """Around 64 queries per compute unit, where the decision kernel starts to
    compute the qualities: embeddings narrower than a slab, a partial last
    slab, whole slabs; ragged last workgroup; with and without the
    per-candidate outputs."""
    import torch
    n = 64 * torch.cuda.get_device_properties(0).multi_processor_count + extra - 63
    sp = S.spec("C2", n_models=7, n_gpu_types=3, hidden=64, embed_dim=embed_dim)
    a = _both(sp, 7, n)
    b = _both(sp, 7, n, candidates=False)
    _same(b, {k: a[k] for k in b})


@pytest.mark.parametrize("n", [200, 1000, 20000])
def test_utilities_without_an_order(n):
    """Infinite and NaN embeddings (qualities, utilities) and bounds that only
    some pairs, or none, meet: a lane's running best, from its first pair at
    -inf to a feasible one, in the small and the streaming form."""
    def edit(qs):
        bits = qs.emb_bits
        bits[0::7, 0] = 0x7F80      # inf
        bits[1::7, 0] = 0xFF80      # -inf
        bits[2::7, 1] = 0x7FC0      # NaN
        bits[3::7, 0] = 0x7F80      # inf - inf in some models
        bits[3::7, 1] = 0x7F80
        qs.slo_s[0::3] = np.float32(0.9)
        qs.slo_s[1::3] = np.float32(1e-30)
    sp = S.spec("C2", n_models=9, n_gpu_types=3, hidden=64, embed_dim=128)
    out = _both(sp, 8, n, edit)
    assert (out["choice"] >= 0).all() and (out["choice"] < 27).all()
    assert 0.0 < out["feasible"].mean() < 1.0


@pytest.mark.parametrize("n", [300, 17001])
@pytest.mark.parametrize("models,gpus", [(1, 1), (2, 1), (7, 1), (5, 3), (16, 1), (17, 1), (21, 3), (32, 2), (13, 5), (31, 3), (16, 8)])
def test_pair_counts(models, gpus, n):
    """Lanes take pairs in steps of 16 and groups of 64: one pair, odd counts on
    both sides of a step and of a group, whole groups; the last pair's
    neighbour in a table row is padding.  Small batches and streaming ones."""
    sp = S.spec("C2", n_models=models, n_gpu_types=gpus, hidden=64, embed_dim=192, gpu_width=8, feat_dim=32)
    kw = dict(cost_weights=[0.0, 0.6, 1.7]) if gpus == 3 else {}
    _both(sp, 9, n, candidates=n < 1000, **kw)


@pytest.mark.parametrize("embed_dim", [128, 192])
def test_streaming_chunks_are_one_launch(embed_dim):
    """A batch whose chunks would each fill the device is routed in one launch:
    the same bits as the staged pipeline in chunks, several tiles to a wave (the
    last one ragged), candidates and qualities included."""
    sp = S.spec("C2", n_models=9, n_gpu_types=3, hidden=64, embed_dim=embed_dim)
    _both(sp, 10, 200_003, max_chunk=16_500)
    r = G.make_router(S.make_problem(sp, 10), max_chunk=16_500)
    r.update(S.make_state(sp, 10))
    r.profile(True)
    G.route_device(r, S.make_queries(sp, 10, n=40_000), "bf16", candidates=False)
    kt = r.profile_read(reset=True)
    r.close()
    assert kt["fused"][1] == 1 and kt["quality"][1] == 0 and kt["mlp"][1] == 1


@pytest.mark.parametrize("embed_dim", [64, 576, 1088])
@pytest.mark.parametrize("n", [20, 1003, 4097, 5000, 9000])
def test_quality_tiles_beside_the_table(embed_dim, n):
    """One, two and three quality tiles to a workgroup (the first two fetched by
    the whole workgroup, 512 k at a time), the last workgroups with few or no
    queries; less than 512 k, a partial second and third."""
    _both(S.spec("C2", n_models=5, n_gpu_types=2, hidden=64, embed_dim=embed_dim), 11, n)
