"""GPU parity of the size-dependent kernel variants at the edges of their
ranges."""
import pytest
import torch

import paper_1908_07341_amd as sd

pytestmark = pytest.mark.gpu

SEED = 777


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sd.lib()


@pytest.mark.parametrize("layout,offset", [(sd.SD_P64, 0), (sd.SD_P64, 8), (sd.SD_I8, 0), (sd.SD_I8, 4)])
@pytest.mark.parametrize("kind,p_up", [(sd.SD_INIT_UP, 0.5), (sd.SD_INIT_DOWN, 0.5), (sd.SD_INIT_RANDOM, 0.5),
                                       (sd.SD_INIT_RANDOM, 0.3), (sd.SD_INIT_RANDOM, 1e-9),
                                       (sd.SD_INIT_RANDOM, 1.0), (sd.SD_INIT_RANDOM, 0.0)])
def test_batch_init_equals_sd_init_per_chain(layout, offset, kind, p_up):
    # one word (8^2), bit strings, whole-word rows and the largest usual size;
    # several words per thread (512^2); the pad between lattices stays as it is
    sizes = [512, 8, 200, 64, 24, 128, 64, 8, 256]
    n = len(sizes)
    print(f"batch init layout={layout} offset={offset} kind={kind} p={p_up}", flush=True)
    plan = sd.sd_batch_plan_create([0.4] * n, [0.6] * n, sizes, [5 * a for a in range(n)], layout=layout, seed=SEED,
                                   k_steps=1, obs_every=0)
    nb = sd.sd_batch_lattice_bytes(plan)
    buf = torch.full((nb + offset,), 0x5A, dtype=torch.uint8, device="cuda")[offset:]
    sd.sd_batch_init(plan, buf, kind, p_up)
    want = torch.full((nb,), 0x5A, dtype=torch.uint8, device="cuda")
    for a, L in enumerate(sizes):
        o = sd.sd_batch_chain_offset(plan, a, 0)
        one = sd.new_lattice(L, layout)
        sd.sd_init(one, L, layout, kind, p_up, SEED, 5 * a)
        flat = one.reshape(-1).view(torch.uint8)
        want[o:o + flat.numel()] = flat
    assert torch.equal(buf, want)
    with pytest.raises(sd.ShakenError):
        sd.sd_batch_init(plan, buf, 7, p_up)
    with pytest.raises(sd.ShakenError):
        sd.sd_batch_init(plan, buf, sd.SD_INIT_RANDOM, 1.5)
    plan.close()
