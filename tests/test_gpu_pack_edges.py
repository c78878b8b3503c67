"""kvprm_pack_kv where the tile count is no multiple of the tiles a block takes at a time (4 at
most): every byte of the layout as the storage contract states it, and no byte past the last tile."""
import pytest
import torch

from gpu_common import kv

pytestmark = pytest.mark.gpu


CASES = [(dt, eb, d, n) for dt, eb in (("f32", 4), ("bf16", 2), ("fp8", 1)) for d in (64, 128)
         for n in (1, 2, 3, 4, 5, 7, 1023)]
# from 128 MiB read and written the tiles go past the caches
CASES += [("bf16", 2, 128, 16387), ("fp8", 1, 64, 65539), ("f32", 4, 64, 16385)]


@pytest.mark.parametrize("dtype,eb,d,ntiles", CASES)
def test_pack_kv_tile_counts(dtype, eb, d, ntiles):
    print(f"case: {dtype} d={d} ntiles={ntiles}", flush=True)
    m = kv()
    gen = torch.Generator().manual_seed(100 * d + ntiles)
    src = torch.randint(0, 256, (ntiles, 16, d, eb), generator=gen, dtype=torch.uint8)
    x, r = 16 // eb, 4 // eb
    want = {m.KVPRM_KEYS: src.reshape(ntiles, 16, d // x, x, eb).transpose(1, 2),
            m.KVPRM_VALUES: src.reshape(ntiles, 4, 4, d // (16 * r), r, 16, eb)
            .permute(0, 3, 1, 5, 4, 2, 6)}
    dev = src.cuda()
    for part, ref in want.items():
        dst = torch.full((ntiles + 1, 16, d, eb), 0xA5, dtype=torch.uint8, device="cuda")
        m.kvprm_pack_kv(dev.data_ptr(), dst.data_ptr(), ntiles, d, dtype, part,
                        torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(dst[:ntiles].cpu().flatten(), ref.reshape(-1))
        assert torch.all(dst[ntiles] == 0xA5)
