"""The attention step at every chunk length its rule can pick (4 to 64 pages; 64 also with all
kv-heads to a block): lengths on both sides of a
chunk's edges, alone and ragged, with and without lengths on the host, against the fp64 oracle, in
exactly the workspace the call asks for.
Bar as in the attention parity tests: 2e-5 of the largest output (fp32 sums, probabilities and
queries in two and three bf16 terms)."""
import numpy as np
import pytest
import torch

import synth
from oracle import inputs as oin
from oracle import kvprm_oracle as ko
from synth.device import DeviceWorkload

from gpu_common import host_activations, kv

pytestmark = pytest.mark.gpu

# heads, kv-heads, d_h, cache dtype, lengths: 4-page chunks of 64 tokens up to 64-page ones
CASES = [
    (28, 4, 128, "bf16", [1]),
    (28, 4, 128, "bf16", [63, 64, 65]),
    # short caches: one launch up to 32 pages and 256 (candidate, kv-head) blocks
    (28, 4, 128, "bf16", [512, 0, 1, 15, 16, 17, 129, 511]),
    (28, 4, 128, "bf16", [513, 3]),
    (32, 2, 128, "fp8", [512, 255, 16, 0, 33]),
    (16, 8, 64, "bf16", [500] + [(37 * i) % 200 for i in range(31)]),
    (16, 8, 64, "fp8", [500] + [(37 * i) % 200 for i in range(32)]),
    (5, 5, 64, "fp8", [65, 512]),
    (12, 12, 64, "f32", [128, 0, 1, 17]),
    (4, 2, 128, "f32", [129, 128, 40]),
    (16, 8, 128, "bf16", [1103]),
    (28, 4, 128, "bf16", [4096, 4033]),
    (28, 4, 128, "bf16", [8192 + 17]),
    (16, 8, 128, "fp8", [511, 0, 2049, 6000, 7001, 3000]),
    (6, 6, 128, "bf16", [2500, 700, 12000]),
    (16, 1, 64, "fp8", [16400]),
    (16, 4, 64, "fp8", [1, 9000, 4097, 0, 129, 6001, 8191, 2048]),
    (32, 2, 128, "bf16", [16384, 16385, 8000, 3]),
    (8, 8, 64, "bf16", [16000] * 8 + [31, 1]),
    (16, 8, 128, "bf16", [4600, 4500]),
    (8, 4, 128, "bf16", [4096] * 13 + [3969, 4095, 2049]),
    (8, 4, 128, "bf16", [1100 - i for i in range(63)] + [0]),
    (16, 8, 128, "bf16", [16000, 31, 15000, 11100]),
    (16, 8, 128, "fp8", [600 * (i % 7) for i in range(64)]),
    (28, 4, 128, "bf16", [30000, 29000, 5, 30001, 29999, 30016, 24000]),
    (4, 4, 128, "bf16", [2049 + i % 40 for i in range(40)] + [0, 70] + [2090 - i for i in range(22)]),
    # very ragged: most candidates without full chunks, the longest first, last and in the middle
    (16, 4, 64, "fp8", [9000 * i * i // 3969 for i in range(64)]),
    (8, 8, 128, "bf16", [14000, 0, 63, 64, 700, 0, 3, 12001, 1, 2999]),
    (8, 2, 64, "bf16", [0] * 31 + [20000] + [0] * 31 + [1]),
]


@pytest.mark.parametrize("nq,nkv,d,dtype,lengths", CASES)
def test_attention_at_every_chunk_length(nq, nkv, d, dtype, lengths):
    print(f"case: nq={nq} nkv={nkv} d={d} {dtype} lengths={lengths}", flush=True)
    shape = synth.ModelShape(1, 256, nq, nkv, d, 256, weight_dtype="f32" if dtype == "f32" else "bf16",
                             kv_dtype=dtype)
    w = synth.make_workload("custom", shape=shape, lengths=lengths, seed=5100 + len(lengths))
    dw = DeviceWorkload(w, nan_unused_pages=True, fill_weights=False)
    q, ks, vs = host_activations(w, 0xABF, scale=1.0)
    ref = ko.attention_layer(shape, oin.cache_from_synth(w), 0, w.lengths, w.page_table,
                             q.astype(np.float64), ks.astype(np.float64), vs.astype(np.float64))
    bar = 2e-5 * max(1.0, float(np.max(np.abs(ref))))
    m = kv()
    qd, kd, vd = (torch.from_numpy(a).cuda() for a in (q, ks, vs))
    st = torch.cuda.current_stream().cuda_stream
    h = m.kvprm_create(dw.desc(m))
    try:
        for host in (True, False):
            batch = dw.batch(m, lengths_host=host)
            n = m.kvprm_workspace_size(h, batch)
            guard = 4096
            ws = torch.full((n + guard,), 0x5A, dtype=torch.uint8, device="cuda")
            o = torch.full(q.shape, float("nan"), device="cuda")

            def call(nbytes):
                m.kvprm_attention(h, dw.cache(m), batch, 0, qd.data_ptr(), kd.data_ptr(),
                                  vd.data_ptr(), ws.data_ptr(), nbytes, o.data_ptr(), st)

            with pytest.raises(m.KvprmError) as e:
                call(n - 1)
            assert e.value.status == m.KVPRM_E_WORKSPACE
            call(n)
            torch.cuda.synchronize()
            got = o.cpu().numpy().astype(np.float64)
            assert np.all(np.isfinite(got)) and torch.all(ws[n:] == 0x5A)
            err = np.max(np.abs(got - ref))
            print(f"  host lengths {host}: max|do| = {err:.2e}", flush=True)
            assert err <= bar
    finally:
        m.kvprm_destroy(h)
