"""The projections of the bf16 pipeline in every form their rules pick, against the fp64 oracle
(section 4.1, Eq. (score)):

* gate/up: one tile pair per block (up to 256 pairs, up to 512 above 16 rows) and, beyond, 2 to 8
  pairs per block with whole and partial last blocks, at 1 to 64 rows (one to eight operand column
  tiles), with and without an adapter's tail, and for inputs that are no whole number of batches;
* q/k/v: the split product and its finish with an adapter on some of q, k and v;
* q/k/v and down on both sides of each limit between the fused and the split form.

Wide models with random weights of a few layers: bars |dP(+)| <= 2e-3 and |dz| <= 2e-2 as in the
parity tests, which a misplaced tile exceeds.

* Precision: an activation's bf16 terms, two of them, three up to four rows. With an empty cache the
  attention is the own value, so the logit's error against fp64 is that of the projections. The
  oracle's pass with every projection's input rounded to two terms gives the error that the terms
  cause by themselves (about 2^-18 of each input); over a few seeds, root mean square, three terms stay
  below half of it and two below twice. (fp32 sums cost about a tenth of it; a lost lo half 2^8 times.)
"""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import inputs as oin
from oracle import kvprm_oracle as ko
from synth.device import DeviceWorkload

from gpu_common import run_score
from test_gpu_lora import _lora_parity

pytestmark = pytest.mark.gpu


def _lengths(B):
    return [(41 * i * i + 5 * i) % 90 for i in range(B)]


def _parity(w):
    p, z = run_score(DeviceWorkload(w, nan_unused_pages=True))
    zr, pr = oin.score_workload(w)
    dp, dz = float(np.max(np.abs(p - pr))), float(np.max(np.abs(z - zr)))
    print(f"  max|dP| = {dp:.3e}  max|dz| = {dz:.3e}", flush=True)
    assert np.all(np.isfinite(z)) and dp <= 2e-3 and dz <= 2e-2


# pairs of gate and up row tiles: the last of one pair per block, then 2, 3, 4, .. 8 per block (8 again
# beyond 2048 pairs), whole and partial last blocks
PAIRS = {256: 1, 260: 2, 512: 2, 516: 3, 520: 3, 772: 4, 1028: 5, 1288: 6, 1540: 7, 1544: 7, 1796: 8, 2052: 8}


@pytest.mark.parametrize("B", [1, 5, 9, 17, 40, 64])
@pytest.mark.parametrize("pairs", PAIRS)
def test_gate_up_pairs(pairs, B):
    print(f"case: {pairs} gate/up pairs, B={B}", flush=True)
    assert min(8, -(-pairs // 256)) == PAIRS[pairs]
    shape = synth.ModelShape(1, 256, 4, 2, 64, 16 * pairs)
    _parity(synth.make_workload("custom", shape=shape, lengths=_lengths(B), seed=8300 + pairs))


@pytest.mark.parametrize("B", [3, 8, 16, 33])
@pytest.mark.parametrize("pairs", [256, 520, 1028])
def test_gate_up_of_an_input_that_is_no_whole_number_of_batches(pairs, B):
    print(f"case: H=192, {pairs} gate/up pairs, B={B}", flush=True)
    shape = synth.ModelShape(1, 192, 4, 2, 64, 16 * pairs)
    _parity(synth.make_workload("custom", shape=shape, lengths=_lengths(B), seed=8400 + pairs))


@pytest.mark.parametrize("B", [4, 12, 20, 48, 64])
@pytest.mark.parametrize("pairs,targets", [(260, synth.LORA_PROJECTIONS), (772, ("gate",)),
                                           (520, ("up", "down"))])
def test_gate_up_adapter_tail(pairs, targets, B):
    print(f"case: {pairs} gate/up pairs, adapter on {targets}, B={B}", flush=True)
    shape = synth.ModelShape(1, 256, 4, 2, 64, 16 * pairs)
    w = synth.make_workload("custom", shape=shape, lengths=_lengths(B), seed=8500 + pairs)
    _lora_parity(w, 64, targets)


@pytest.mark.parametrize("B", [9, 17, 40, 64])
@pytest.mark.parametrize("targets", [("q", "v"), ("k",), ("q", "k", "v", "o")])
def test_split_qkv_adapter_tail(targets, B):
    """64 / 8 heads of 128: 320 rotary tile pairs, more than the fused kernel takes."""
    print(f"case: split q/k/v, adapter on {targets}, B={B}", flush=True)
    shape = synth.ModelShape(1, 256, 64, 8, 128, 512)
    w = synth.make_workload("custom", shape=shape, lengths=_lengths(B), seed=8600 + B)
    _lora_parity(w, 96, targets)


@pytest.mark.parametrize("H,F,B", [
    (256, 2048, 1), (256, 2304, 5), (512, 4096, 8), (512, 4608, 3), (2048, 8192, 4), (2048, 8704, 8),
    (256, 2048, 9), (256, 2176, 16), (320, 1024, 17), (320, 1152, 64),   # down
    (2944, 512, 17), (3072, 512, 33), (3072, 512, 16), (3072, 512, 64)])  # q/k/v
def test_each_side_of_the_split_limits(H, F, B):
    print(f"case: H={H} F={F} B={B}", flush=True)
    shape = synth.ModelShape(2, H, 4, 2, 64, F)
    _parity(synth.make_workload("custom", shape=shape, lengths=_lengths(B), seed=8650 + B))


def _bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32).astype(np.float64)


def _two_terms(x):
    hi = _bf16(x)
    return hi + _bf16(x - hi)


def _logit_of_empty_cache(w, rnd):
    """The oracle's pass for a candidate without cached tokens, the inputs of the projections passed
    through rnd (gain applied before, RMSNorm scale after the product, as the kernels do)."""
    s, ro = w.shape, oin.readout_from_synth(w.shape, w.seed)
    scale = lambda x: 1.0 / np.sqrt(np.mean(x * x) + s.rms_eps)
    x = np.array(ro.verify_embed, np.float64)
    for l in range(s.num_layers):
        W = ro.layer(l)
        v = (W.wv @ rnd(x * W.attn_norm) * scale(x)).reshape(s.num_kv_heads, s.head_dim)
        x = x + W.wo @ rnd(np.repeat(v, s.num_q_heads // s.num_kv_heads, axis=0).ravel())
        u, r = rnd(x * W.ffn_norm), scale(x)
        x = x + W.w_down @ rnd(ko.silu(W.w_gate @ u * r) * (W.w_up @ u * r))
    return float(ro.reward_w @ (x * scale(x) * ro.final_norm))


@pytest.mark.parametrize("shape", [synth.ModelShape(2, 512, 8, 2, 64, 1024),      # fused projections
                                   synth.ModelShape(2, 512, 64, 8, 128, 4352)])   # split ones
def test_terms_of_the_activations(shape):
    seeds = range(8700, 8712)
    err = {B: [] for B in (1, 3, 4, 5, 8, 9)}
    terms = []
    for seed in seeds:
        for B in err:
            w = synth.make_workload("custom", shape=shape, lengths=[0] * B, seed=seed)
            z = run_score(DeviceWorkload(w))[1]
            if B == 1:
                zr = oin.score_workload(w)[0][0]
                assert abs(_logit_of_empty_cache(w, lambda x: x) - zr) <= 1e-12 * max(1.0, abs(zr))
                terms.append(_logit_of_empty_cache(w, _two_terms) - zr)
            err[B].append(z - zr)
    two = float(np.sqrt(np.mean(np.square(terms))))
    print(f"case: H={shape.hidden}, two terms alone {two:.2e}", flush=True)
    for B, e in err.items():
        rows = np.sqrt(np.mean(np.square(e), axis=0))  # of every row
        print(f"  B={B}: rms error of the rows {rows.min():.2e} .. {rows.max():.2e}", flush=True)
        assert rows.max() <= (0.5 if B <= 4 else 2.0) * two, B
