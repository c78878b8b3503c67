"""The workspace sizes never fall when a batch grows, in candidates or in page-table width, with any
of the readout's options: a workspace sized for the largest batch serves every smaller one."""
import pytest

import paper_2607_09153_amd as kv

FAKE = 4096
SHAPES = [(28, 3584, 28, 4, 128, 18944), (28, 1024, 16, 8, 128, 3072), (2, 256, 4, 2, 64, 1024),
          (2, 2048, 32, 2, 128, 2048)]


@pytest.mark.parametrize("wdt,kvdt", [("bf16", "bf16"), ("bf16", "fp8"), ("f32", "f32")])
@pytest.mark.parametrize("shape", SHAPES)
def test_workspace_never_falls(shape, wdt, kvdt):
    h = kv.kvprm_create(kv.make_desc(*shape, weight_dtype=wdt, kv_dtype=kvdt))
    calls = [(kv.kvprm_workspace_size, (1, 2, 3, 7, 8, 9, 16, 17, 33, 34, 64))]
    if kvdt == "bf16":
        calls.append((kv.kvprm_workspace_size_grad, range(1, 9)))
    if wdt == "bf16":
        for rank in (32, 256, 512):
            calls.append((lambda h, b, r=rank: kv.kvprm_workspace_size_lora(h, b, r), calls[0][1]))
        for depth in (2, 3, 4, 8):
            if depth * shape[2] // shape[3] <= 16:
                size = lambda h, b, o=kv.make_options(depth=depth): kv.kvprm_workspace_size_ex(h, b, o)
                calls.append((size, [B for B in calls[0][1] if B * depth <= 64]))
    try:
        for size, batches in calls:
            last = {}
            for B in batches:
                row = 0
                for pages in (1, 2, 5, 16, 17, 33, 69, 128, 300, 512, 1000, 2048):
                    n = size(h, kv.make_batch(B, FAKE, pages, FAKE))
                    assert n >= row and n >= last.get(pages, 0), (B, pages)
                    row = last[pages] = n
    finally:
        kv.kvprm_destroy(h)
