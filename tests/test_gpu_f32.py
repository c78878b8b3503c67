"""The fp32 pipeline at the edges of its launches, against the fp64 oracle: 16, 32 and 64 candidates
to a projection block and one more than that (and several blocks of them), inputs that leave waves
of a block without work, kv-heads beyond the bf16 limit, chunks of 2 to 32 pages. Bars as in the
parity tests with fp32 weights: |dP(+)| <= 1e-5, |dz| <= 4e-5."""
import numpy as np
import pytest

import synth
from oracle import inputs as oin
from synth.device import DeviceWorkload

from gpu_common import run_score

pytestmark = pytest.mark.gpu

# layers, hidden, q-heads, kv-heads, d_h, ffn, lengths
CASES = [
    (2, 64, 1, 1, 64, 64, [33]),
    (2, 192, 12, 12, 64, 320, [0, 1, 700]),
    (1, 256, 16, 1, 128, 192, [31 * (i + 1) for i in range(16)]),
    (1, 256, 4, 2, 64, 512, [(37 * i) % 300 for i in range(17)]),
    (1, 320, 6, 3, 64, 256, [(53 * i) % 200 for i in range(33)]),
    (1, 128, 2, 1, 128, 128, [(29 * i) % 130 for i in range(65)]),
    (1, 64, 2, 2, 64, 128, [(31 * i) % 90 for i in range(130)]),
    (1, 256, 4, 2, 64, 256, [9000, 4097, 16000]),
]


@pytest.mark.parametrize("layers,H,nq,nkv,d,F,lengths", CASES)
def test_f32_pipeline(layers, H, nq, nkv, d, F, lengths):
    print(f"case: layers={layers} H={H} nq={nq} nkv={nkv} d={d} F={F} B={len(lengths)}", flush=True)
    shape = synth.ModelShape(layers, H, nq, nkv, d, F, weight_dtype="f32", kv_dtype="f32")
    w = synth.make_workload("custom", shape=shape, lengths=lengths, seed=5200 + len(lengths))
    dw = DeviceWorkload(w, nan_unused_pages=True)
    z_ref, p_ref = oin.score_workload(w)
    for host in (True, False):
        p, z = run_score(dw, lengths_host=host)
        dp, dz = np.max(np.abs(p - p_ref)), np.max(np.abs(z - z_ref))
        print(f"  host lengths {host}: max|dP| = {dp:.2e}, max|dz| = {dz:.2e}", flush=True)
        assert np.all(np.isfinite(z)) and dp <= 1e-5 and dz <= 4e-5
