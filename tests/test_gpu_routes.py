"""GPU parity of the size-dependent kernel variants at the edges of their
ranges."""
import ctypes
import json
import threading

import numpy as np
import pytest
import torch

import paper_1908_07341_amd as sd
from paper_1908_07341_amd import inputs

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


@pytest.mark.parametrize("layout", [sd.SD_P64, sd.SD_I8])
def test_captured_batch_init_outlives_its_plan(layout):
    # the graph holds the caller's lattices and nothing of the plan, whose
    # device tables are freed, and their memory used again, before the replays
    sizes = [64, 200, 8, 64]
    plan = sd.sd_batch_plan_create([0.4] * 4, [0.6] * 4, sizes, [3 * a for a in range(4)], layout=layout, seed=SEED, k_steps=1,
                                   obs_every=0)
    nb = sd.sd_batch_lattice_bytes(plan)
    want = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    sd.sd_batch_init(plan, want, sd.SD_INIT_RANDOM, 0.3)
    buf = torch.zeros_like(want)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        sd.sd_batch_init(plan, buf, sd.SD_INIT_RANDOM, 0.3)
    plan.close()
    other = sd.sd_batch_plan_create([0.1] * 4, [0.2] * 4, sizes[::-1], [50 + a for a in range(4)], layout=layout, seed=1,
                                    k_steps=1, obs_every=0)
    for _ in range(3):
        buf.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(buf, want)
    other.close()


@pytest.mark.parametrize("L", [7, 8, 9, 11, 31, 63, 65, 127, 333])
@pytest.mark.parametrize("offset", [0, 1])
def test_int8_windows(oracle, L, offset):
    # lattices of one word and less (7, 8), rows shorter than a word, rows whose
    # wrap falls on every bit of a word, a last word of any length, and
    # neighbour windows across the lattice's end; any address
    print(f"int8 windows L={L} offset={offset}", flush=True)
    lat = inputs.random_lattice(L, L)
    buf = torch.zeros(2 * (L * L + 16), dtype=torch.int8, device="cuda")
    src = buf[offset:offset + L * L]
    dst = buf[L * L + 16 - (16 - offset) % 16:][:L * L]
    for which in (0, 1):
        src.copy_(torch.from_numpy(lat.reshape(-1)))
        sd.sd_half_step(src, dst, L, sd.SD_I8, which, 0.4, 0.9, SEED, 3, 6 + which)
        want = oracle.half_step(lat, 0.4, 0.9, which, SEED, 3, 6 + which)
        assert np.array_equal(dst.cpu().numpy().reshape(L, L), want)
        assert np.array_equal(src.cpu().numpy().reshape(L, L), lat)


@pytest.mark.parametrize("L,layout", [(6784, sd.SD_P64), (6848, sd.SD_P64), (8192, sd.SD_P64), (6848, sd.SD_P32),
                                      (6720, sd.SD_P32), (14144, sd.SD_P64), (14208, sd.SD_P64), (19904, sd.SD_P64)])
def test_wide_and_one_word_tiles_agree(L, layout):
    # below and above the size from which packed lattices take wide tiles, and
    # those from which they take more workgroups; the runs of sd_run_many too
    # short for whole steps take one-word tiles
    print(f"tiles L={L} layout={layout}", flush=True)
    lat = [sd.new_lattice(L, layout) for _ in range(4)]
    for x in (lat[0], lat[2]):
        sd.sd_init(x, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    obs = torch.empty((2, 2, 3), dtype=torch.int64, device="cuda")
    sd.sd_run(lat[0], lat[1], L, layout, 0.5, 0.5, SEED, 1, 0, 2, obs[0], 1)
    sd.sd_run_many([lat[2]], [lat[3]], L, layout, [0.5], [0.5], SEED, [1], 0, 2, obs[1], 1)
    assert torch.equal(lat[0], lat[2]) and torch.equal(lat[1], lat[3]) and torch.equal(obs[0], obs[1])


@pytest.mark.parametrize("L,layout", [(100, sd.SD_I8), (200, sd.SD_P64), (576, sd.SD_P64)])
def test_records_of_one_word_tiles_under_capture(oracle, L, layout):
    # no partial-sum buffer can be made on a stream first used under capture:
    # the records come from atomics, and every replay writes the same ones
    print(f"capture L={L} layout={layout}", flush=True)
    sigma, tau = sd.new_lattice(L, layout), sd.new_lattice(L, layout)
    start = inputs.random_lattice(L, 5)
    host = start if layout == sd.SD_I8 else inputs.pack_bits(start)
    first = torch.from_numpy(host.reshape(-1).copy()).cuda()
    flat = sigma.reshape(-1).view(torch.int8 if layout == sd.SD_I8 else torch.uint8)
    obs = torch.empty((3, 3), dtype=torch.int64, device="cuda")
    _, _, want = oracle.run(start, 0.4, 0.6, SEED, 2, 0, 3, obs_every=1)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        flat.copy_(first)
        sd.sd_run(sigma, tau, L, layout, 0.4, 0.6, SEED, 2, 0, 3, obs, 1, sd.SD_FLAG_GLOBAL_KERNELS)
    for _ in range(3):
        obs.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(obs.cpu().numpy(), want)


@pytest.mark.parametrize("L", [8, 16, 24, 32, 40, 48, 56, 64])
@pytest.mark.parametrize("J,q", [(0.4, 0.6), (0.0, 0.0), (0.5, 1.0), (-0.7, 0.3), (9.0, 20.0)])
def test_small_lattices_drawn_ahead(oracle, L, J, q):
    # every side of the small-lattice kernel: one row, two rows and other
    # fractions of a row per word; runs of one step, below, at and past the
    # half-steps drawn ahead at a time (14 at 64^2, 64 at 8^2), several rounds
    # with a ragged end; thresholds with equal top bytes (0, 0), with no tail
    # (h = 0) and at the ends of their range.  The grid kernels are the general
    # path; the shortest and a middle run also go through the oracle.
    print(f"small L={L} J={J} q={q}", flush=True)
    start = inputs.random_lattice(L, 3 * L)
    for layout in (sd.SD_P64, sd.SD_I8, sd.SD_P32):
        if layout == sd.SD_P32 and L % 32:
            continue
        host = start if layout == sd.SD_I8 else inputs.pack_bits(start)
        host = torch.from_numpy(host.reshape(-1).copy()).cuda()
        for k, every, flags in [(1, 1, 0), (6, 1, 0), (7, 2, 0), (8, 1, sd.SD_FLAG_COMPLEMENT_RNG), (32, 3, 0), (33, 1, 0),
                                (150, 7, 0), (5, 0, 0)]:
            got = []
            for f in (flags, flags | sd.SD_FLAG_GLOBAL_KERNELS):
                # int8 lattices at an odd address, words at their own alignment
                pad = 1 if layout == sd.SD_I8 else 8
                buf = torch.full((2, host.numel() + 64), 3, dtype=host.dtype, device="cuda")
                sigma, tau = buf[0, pad:pad + host.numel()], buf[1, pad:pad + host.numel()]
                sigma.copy_(host)
                obs = torch.full((k // every if every else 0, 3), -1, dtype=torch.int64, device="cuda")
                sd.sd_run(sigma, tau, L, layout, J, q, SEED, 4, 11, k, obs if every else None, every, f)
                got.append((buf, obs))
            assert torch.equal(got[0][0], got[1][0]), (layout, k)
            assert torch.equal(got[0][1], got[1][1]), (layout, k)
            if k in (1, 33):
                sig, tau, rec = oracle.run(start, J, q, SEED, 4, 11, k, obs_every=every)
                flat = got[0][0][0, pad:pad + host.numel()].cpu().numpy()
                have = flat.reshape(L, L) if layout == sd.SD_I8 else inputs.unpack_bits(flat, L)
                assert np.array_equal(have, sig) and np.array_equal(got[0][1].cpu().numpy(), rec)


@pytest.mark.parametrize("L", [8, 32, 48, 64])
def test_exact_samples_shared_and_alone(oracle, L):
    # more pairs than CUs (two workgroups share a CU) against
    # the same pairs alone (16 wavefronts), and one pair against the oracle;
    # at T_max = 16 most pairs stay open
    J, q, n = 0.3, 0.8, 300
    print(f"exact samples L={L}", flush=True)
    nb = sd.sd_lattice_bytes(L, sd.SD_P64)
    for T0, T_max in ((16, 4096), (1, 16)):
        out = torch.full((n, nb), 9, dtype=torch.uint8, device="cuda")
        work = torch.empty(4 * n * nb, dtype=torch.uint8, device="cuda")
        T = sd.sd_propp_wilson(out, work, n, L, J, q, SEED, 50, 1 << 20, T0, T_max)
        one = torch.full((7, nb), 9, dtype=torch.uint8, device="cuda")
        T1 = sd.sd_propp_wilson(one, work, 7, L, J, q, SEED, 60, 1 << 20, T0, T_max)
        assert T[10:17] == T1
        assert torch.equal(out[10:17], one)
        want, t = oracle.propp_wilson(L, J, q, SEED, 60, 1 << 20, T0, T_max)
        assert t == T1[0]
        assert np.array_equal(inputs.unpack_bits(one[0].cpu().numpy(), L), want)


@pytest.mark.parametrize("L,layout,k,every", [
    (8, sd.SD_P64, 1100, 1), (9, sd.SD_I8, 40, 1), (32, sd.SD_P32, 300, 7), (64, sd.SD_I8, 700, 1), (63, sd.SD_I8, 20, 2),
    (65, sd.SD_I8, 33, 1), (72, sd.SD_P64, 1, 1), (127, sd.SD_I8, 5, 0), (128, sd.SD_P64, 90, 3), (160, sd.SD_P32, 9, 1),
    (181, sd.SD_I8, 12, 1), (182, sd.SD_I8, 12, 1), (192, sd.SD_P64, 150, 4), (200, sd.SD_P64, 150, 1), (256, sd.SD_I8, 200, 1),
    (257, sd.SD_I8, 30, 1), (320, sd.SD_P64, 100, 1), (360, sd.SD_P64, 64, 5), (362, sd.SD_I8, 70, 1), (363, sd.SD_I8, 3, 1)])
def test_drawn_ahead_by_the_device(L, layout, k, every):
    # every form of the walker (rows in registers, whole words, bit strings; one
    # and two words a thread; partial last words), the sizes where they change
    # hands, one round and several with a ragged last one, records of rounds
    # that end between two of them; against the grid kernels
    print(f"ahead L={L} layout={layout} k={k}", flush=True)
    start = sd.new_lattice(L, layout)
    sd.sd_init(start, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    for flags in (0, sd.SD_FLAG_COMPLEMENT_RNG):
        got = []
        for f in (flags, flags | sd.SD_FLAG_GLOBAL_KERNELS):
            sigma, tau = start.clone(), torch.zeros_like(start)
            obs = torch.full((k // every if every else 0, 3), -1, dtype=torch.int64, device="cuda")
            sd.sd_run(sigma, tau, L, layout, 0.45, 0.9, SEED, 8, 5, k, obs if every else None, every, f)
            got.append((sigma, tau, obs))
        for a, b in zip(*got):
            assert torch.equal(a, b)


@pytest.mark.parametrize("L,layout,n", [(16, sd.SD_P64, 16), (64, sd.SD_I8, 3), (100, sd.SD_I8, 5), (200, sd.SD_P64, 2),
                                        (256, sd.SD_I8, 16), (320, sd.SD_P32, 3)])
def test_several_chains_drawn_ahead(L, layout, n):
    # chains of different couplings and streams share a launch; each is its own sd_run
    print(f"several chains ahead L={L} n={n}", flush=True)
    k, every = 40, 3
    J, q, streams = [0.2 + 0.1 * a for a in range(n)], [1.5 - 0.1 * a for a in range(n)], [7 * a + 1 for a in range(n)]
    sig, tau = [], []
    for a in range(n):
        x = sd.new_lattice(L, layout)
        sd.sd_init(x, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, a)
        sig.append(x)
        tau.append(torch.zeros_like(x))
    first = [x.clone() for x in sig]
    obs = torch.full((n, k // every, 3), -1, dtype=torch.int64, device="cuda")
    sd.sd_run_many(sig, tau, L, layout, J, q, SEED, streams, 3, k, obs, every)
    for a in range(n):
        one, two = first[a].clone(), torch.zeros_like(first[a])
        rec = torch.empty((k // every, 3), dtype=torch.int64, device="cuda")
        sd.sd_run(one, two, L, layout, J[a], q[a], SEED, streams[a], 3, k, rec, every, sd.SD_FLAG_GLOBAL_KERNELS)
        assert torch.equal(one, sig[a]) and torch.equal(two, tau[a]) and torch.equal(rec, obs[a])


@pytest.mark.parametrize("L,layout,k,route", [
    (8, sd.SD_P64, 1100, sd.SD_ROUTE_AHEAD), (8, sd.SD_P64, 1000, sd.SD_ROUTE_SMALL), (32, sd.SD_P32, 300, sd.SD_ROUTE_AHEAD),
    (32, sd.SD_P64, 63, sd.SD_ROUTE_SMALL), (64, sd.SD_I8, 16, sd.SD_ROUTE_AHEAD), (64, sd.SD_I8, 15, sd.SD_ROUTE_SMALL),
    (9, sd.SD_I8, 40, sd.SD_ROUTE_AHEAD), (65, sd.SD_I8, 33, sd.SD_ROUTE_AHEAD), (136, sd.SD_P64, 30, sd.SD_ROUTE_AHEAD),
    (360, sd.SD_P64, 20, sd.SD_ROUTE_AHEAD), (362, sd.SD_I8, 20, sd.SD_ROUTE_AHEAD), (363, sd.SD_I8, 3, sd.SD_ROUTE_HALF_STEPS),
    (368, sd.SD_P64, 3, sd.SD_ROUTE_HALF_STEPS), (384, sd.SD_P64, 3, sd.SD_ROUTE_BANDS), (384, sd.SD_I8, 2, sd.SD_ROUTE_HALF_STEPS),
    (4096, sd.SD_P64, 3, sd.SD_ROUTE_BANDS), (4160, sd.SD_P64, 3, sd.SD_ROUTE_HALF_STEPS)])
def test_route_by_size(L, layout, k, route):
    # the kernels that the runs of the tests around this one take, at the sizes
    # where they change hands
    print(f"route L={L} layout={layout} k={k}", flush=True)
    sigma, tau = sd.new_lattice(L, layout), sd.new_lattice(L, layout)
    sd.sd_init(sigma, L, layout, sd.SD_INIT_UP)
    sd.sd_run(sigma, tau, L, layout, 0.4, 0.6, SEED, 1, 0, k)
    assert sd.sd_debug_last_route() == route
    if route != sd.SD_ROUTE_SMALL:   # a call of several chains has no route of its own for short runs
        sd.sd_run_many([sigma], [tau], L, layout, [0.4], [0.6], SEED, [1], 0, k)
        assert sd.sd_debug_last_route() == route
    sd.sd_run(sigma, tau, L, layout, 0.4, 0.6, SEED, 1, 0, k, None, 0, sd.SD_FLAG_GLOBAL_KERNELS)
    assert sd.sd_debug_last_route() == sd.SD_ROUTE_HALF_STEPS
    with pytest.raises(sd.ShakenError):
        sd.sd_run(sigma, sigma, L, layout, 0.4, 0.6, SEED, 1, 0, k)
    assert sd.sd_debug_last_route() == sd.SD_ROUTE_NONE


def test_more_streams_than_scratch_buffers():
    # the scratch of drawn-ahead runs is made for a bounded number of streams;
    # runs on further ones take other kernels and give the same chains
    L, k = 96, 30
    start = sd.new_lattice(L, sd.SD_P64)
    sd.sd_init(start, L, sd.SD_P64, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    torch.cuda.synchronize()
    out = []
    streams = [torch.cuda.Stream() for _ in range(20)]
    for st in streams:
        sigma, tau = start.clone(), torch.zeros_like(start)
        obs = torch.zeros((k, 3), dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        sd.sd_run(sigma, tau, L, sd.SD_P64, 0.4, 0.6, SEED, 1, 0, k, obs, 1, hip_stream=st)
        out.append((sigma, tau, obs))
    torch.cuda.synchronize()
    for o in out[1:]:
        assert all(torch.equal(x, y) for x, y in zip(o, out[0]))


def test_every_stream_draws_ahead():
    # more streams than scratch buffers, busy at the same time with chains of
    # their own, destroyed and made anew: all draw ahead, and no run takes another's buffer
    L, k, n = 200, 40, 24
    first = sd.new_lattice(L, sd.SD_P64)
    sd.sd_init(first, L, sd.SD_P64, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    hip = ctypes.CDLL("libamdhip64.so")

    def new():
        return first.clone(), torch.zeros_like(first), torch.full((k, 3), -1, dtype=torch.int64, device="cuda")

    want = [new() for _ in range(n)]
    for i, w in enumerate(want):
        sd.sd_run(w[0], w[1], L, sd.SD_P64, 0.4, 0.6, SEED, i, 0, k, w[2], 1, sd.SD_FLAG_GLOBAL_KERNELS)
    for _ in range(2):
        streams = [ctypes.c_void_p() for _ in range(n)]
        for s in streams:
            assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        got = [[new() for _ in range(3)] for _ in range(n)]
        torch.cuda.synchronize()
        for r in range(3):
            for i, s in enumerate(streams):
                g = got[i][r]
                sd.sd_run(g[0], g[1], L, sd.SD_P64, 0.4, 0.6, SEED, i, 0, k, g[2], 1, hip_stream=s.value)
                assert sd.sd_debug_last_route() == sd.SD_ROUTE_AHEAD, i
        torch.cuda.synchronize()
        for i, s in enumerate(streams):
            assert all(torch.equal(a, b) for g in got[i] for a, b in zip(g, want[i])), i
            assert hip.hipStreamDestroy(s) == 0


def test_tuned_choices_of_other_kernel_sets_are_measured_again(tmp_path):
    # an entry that an earlier library left (one launch per half-step, 16
    # workgroups for 256-word tiles) is no choice among the present kernels
    L, layout, path = 768, sd.SD_P64, str(tmp_path / "tune.json")
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    old = 2 | (16 << 3) | (4 << 24)
    with open(path, "w") as f:
        json.dump({f"run:{arch}:L={L}:layout={layout}": old}, f)
    sd.sd_tune(L, layout, path)
    mode, _, blocks, _ = sd.sd_tuned_choice(L, layout)
    assert (mode, blocks) != (2, 16)
    entries = json.load(open(path))
    assert entries[f"run:{arch}:L={L}:layout={layout}"] == old   # left to the library that wrote it
    assert f"run2:{arch}:L={L}:layout={layout}" in entries


@pytest.mark.parametrize("L,layout,route", [(64, sd.SD_P64, sd.SD_ROUTE_SMALL), (192, sd.SD_P64, sd.SD_ROUTE_LDS),
                                            (256, sd.SD_P64, sd.SD_ROUTE_LDS), (200, sd.SD_P64, sd.SD_ROUTE_LDS),
                                            (320, sd.SD_P64, sd.SD_ROUTE_BANDS), (101, sd.SD_I8, sd.SD_ROUTE_HALF_STEPS)])
def test_tuned_runs_without_scratch(tmp_path, L, layout, route):
    # sizes that draw ahead when they can: runs that cannot (no allocation, or
    # captured) are tuned among the kernels that they can take, and the eager
    # runs stay drawn ahead; sixteen tiles of 256^2 want eight wavefronts
    print(f"tuned without scratch L={L} layout={layout}", flush=True)
    path, k = str(tmp_path / "tune.json"), 20
    sd.sd_tune(L, layout, path)
    choice = sd.sd_tuned_choice(L, layout)
    print("tuned", choice, open(path).read(), flush=True)
    assert choice[0] == 1
    if L == 256:
        assert choice[3] == 512
    first = sd.new_lattice(L, layout)
    sd.sd_init(first, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    out = []
    for run, flags, want in ((sd.sd_run, 0, sd.SD_ROUTE_AHEAD), (sd.sd_run_noalloc, 0, route),
                             (sd.sd_run, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS)):
        sigma, tau = first.clone(), torch.zeros_like(first)
        obs = torch.full((k, 3), -1, dtype=torch.int64, device="cuda")
        run(sigma, tau, L, layout, 0.4, 0.6, SEED, 1, 0, k, obs, 1, flags)
        assert sd.sd_debug_last_route() == want
        out.append((sigma, tau, obs))
    for o in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, out[0]))
    sd.sd_tune(L, layout, path)   # from the cache
    assert sd.sd_tuned_choice(L, layout) == choice


@pytest.mark.parametrize("L,layout,k,every,route,many", [
    (64, sd.SD_I8, 1, 1, sd.SD_ROUTE_SMALL, sd.SD_ROUTE_AHEAD), (33, sd.SD_I8, 1, 1, sd.SD_ROUTE_AHEAD, sd.SD_ROUTE_AHEAD),
    (72, sd.SD_P64, 1, 1, sd.SD_ROUTE_LDS, sd.SD_ROUTE_AHEAD), (88, sd.SD_P64, 1, 0, sd.SD_ROUTE_LDS, sd.SD_ROUTE_AHEAD),
    (181, sd.SD_I8, 1, 1, sd.SD_ROUTE_AHEAD, sd.SD_ROUTE_AHEAD), (182, sd.SD_I8, 1, 1, sd.SD_ROUTE_HALF_STEPS, sd.SD_ROUTE_HALF_STEPS),
    (128, sd.SD_I8, 2, 1, sd.SD_ROUTE_LDS, sd.SD_ROUTE_AHEAD), (128, sd.SD_I8, 2, 0, sd.SD_ROUTE_AHEAD, sd.SD_ROUTE_AHEAD),
    (136, sd.SD_P64, 2, 1, sd.SD_ROUTE_AHEAD, sd.SD_ROUTE_AHEAD), (96, sd.SD_P32, 2, 1, sd.SD_ROUTE_AHEAD, sd.SD_ROUTE_AHEAD),
    (248, sd.SD_P64, 1, 1, sd.SD_ROUTE_LDS, sd.SD_ROUTE_HALF_STEPS), (360, sd.SD_P64, 1, 1, sd.SD_ROUTE_HALF_STEPS, sd.SD_ROUTE_HALF_STEPS),
    (333, sd.SD_I8, 1, 0, sd.SD_ROUTE_HALF_STEPS, sd.SD_ROUTE_HALF_STEPS)])
def test_short_runs(oracle, L, layout, k, every, route, many):
    # runs too short to be drawn ahead, on each side of the rule
    print(f"short run L={L} layout={layout} k={k} every={every}", flush=True)
    start = inputs.random_lattice(L, L)
    host = start if layout == sd.SD_I8 else inputs.pack_bits(start)
    host = torch.from_numpy(host.reshape(-1).copy()).cuda()
    sig, tau, rec = oracle.run(start, 0.4, 0.7, SEED, 3, 5, k, obs_every=every)
    for call, want in (("run", route), ("many", many)):
        sigma, t = sd.new_lattice(L, layout), sd.new_lattice(L, layout)
        flat = [x.reshape(-1).view(host.dtype) for x in (sigma, t)]
        flat[0].copy_(host)
        obs = torch.full((k // every if every else 0, 3), -1, dtype=torch.int64, device="cuda")
        if call == "run":
            sd.sd_run(sigma, t, L, layout, 0.4, 0.7, SEED, 3, 5, k, obs if every else None, every)
        else:
            sd.sd_run_many([sigma], [t], L, layout, [0.4], [0.7], SEED, [3], 5, k, obs if every else None, every)
        assert sd.sd_debug_last_route() == want, call
        for x, w in zip(flat, (sig, tau)):
            have = x.cpu().numpy()
            assert np.array_equal(have.reshape(L, L) if layout == sd.SD_I8 else inputs.unpack_bits(have, L), w), call
        if every:
            assert np.array_equal(obs.cpu().numpy(), rec), call


@pytest.mark.parametrize("L,layout,n,k,every,route", [
    (320, sd.SD_P64, 8, 10, 3, sd.SD_ROUTE_AHEAD), (320, sd.SD_P64, 9, 10, 3, sd.SD_ROUTE_BANDS), (320, sd.SD_I8, 16, 9, 2, sd.SD_ROUTE_AHEAD),
    (320, sd.SD_I8, 16, 10, 2, sd.SD_ROUTE_BANDS), (360, sd.SD_P64, 16, 11, 1, sd.SD_ROUTE_AHEAD), (362, sd.SD_I8, 16, 13, 4, sd.SD_ROUTE_AHEAD),
    (361, sd.SD_I8, 15, 7, 0, sd.SD_ROUTE_AHEAD), (256, sd.SD_P64, 16, 21, 5, sd.SD_ROUTE_AHEAD)])
def test_many_chains_of_the_largest_drawn_ahead(oracle, L, layout, n, k, every, route):
    # as many chains as leave rounds of four to ten half-steps, which end between
    # records and in the middle of a ragged last round, and on each side of the
    # rule that sends rows of whole words to the bands; the first and last chain
    # against the oracle
    print(f"many chains L={L} layout={layout} n={n} k={k}", flush=True)
    J, q, ids = [0.2 + 0.05 * a for a in range(n)], [1.2 - 0.05 * a for a in range(n)], [3 * a + 1 for a in range(n)]
    starts = [inputs.random_lattice(L, 100 + a) for a in range(n)]
    sig, tau = [], []
    for x in starts:
        host = x if layout == sd.SD_I8 else inputs.pack_bits(x)
        t = sd.new_lattice(L, layout)
        t.reshape(-1).view(torch.int8 if layout == sd.SD_I8 else torch.uint8).copy_(torch.from_numpy(host.reshape(-1).copy()))
        sig.append(t)
        tau.append(torch.zeros_like(t))
    obs = torch.full((n, k // every if every else 0, 3), -1, dtype=torch.int64, device="cuda")
    sd.sd_run_many(sig, tau, L, layout, J, q, SEED, ids, 2, k, obs if every else None, every)
    assert sd.sd_debug_last_route() == route

    def host(t):
        flat = t.cpu().numpy().reshape(-1)
        return flat.reshape(L, L) if layout == sd.SD_I8 else inputs.unpack_bits(flat.view(np.uint8), L)

    for a in (0, n - 1):
        s, t, rec = oracle.run(starts[a], J[a], q[a], SEED, ids[a], 2, k, obs_every=every)
        assert np.array_equal(host(sig[a]), s) and np.array_equal(host(tau[a]), t), a
        if every:
            assert np.array_equal(obs[a].cpu().numpy(), rec), a


@pytest.mark.parametrize("L,layout,k,every,flags,route", [
    (32, sd.SD_P32, 300, 7, 0, sd.SD_ROUTE_AHEAD), (64, sd.SD_I8, 130, 1, 0, sd.SD_ROUTE_AHEAD), (33, sd.SD_I8, 40, 3, 0, sd.SD_ROUTE_AHEAD),
    (128, sd.SD_P64, 300, 11, 0, sd.SD_ROUTE_AHEAD), (100, sd.SD_I8, 50, 1, 0, sd.SD_ROUTE_AHEAD), (150, sd.SD_I8, 40, 2, 0, sd.SD_ROUTE_AHEAD),
    (192, sd.SD_P64, 60, 5, 0, sd.SD_ROUTE_AHEAD), (200, sd.SD_P64, 60, 1, 0, sd.SD_ROUTE_AHEAD), (256, sd.SD_I8, 40, 1, 0, sd.SD_ROUTE_AHEAD),
    (320, sd.SD_P64, 45, 4, 0, sd.SD_ROUTE_AHEAD), (333, sd.SD_I8, 45, 1, 0, sd.SD_ROUTE_AHEAD), (384, sd.SD_P64, 20, 3, 0, sd.SD_ROUTE_BANDS),
    (448, sd.SD_I8, 11, 1, 0, sd.SD_ROUTE_BANDS), (704, sd.SD_P64, 9, 2, 0, sd.SD_ROUTE_BANDS), (2112, sd.SD_P64, 4, 1, 0, sd.SD_ROUTE_BANDS),
    (100, sd.SD_I8, 5, 1, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS), (333, sd.SD_I8, 5, 1, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS),
    (200, sd.SD_P64, 5, 1, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS), (448, sd.SD_I8, 3, 1, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS),
    (96, sd.SD_P32, 5, 1, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS), (704, sd.SD_P64, 3, 1, sd.SD_FLAG_GLOBAL_KERNELS, sd.SD_ROUTE_HALF_STEPS)])
def test_every_form_against_the_oracle(oracle, L, layout, k, every, flags, route):
    # each form of the walker, the bands and the one-word tiles that the tests
    # around this one compare with each other, once against the oracle
    print(f"form L={L} layout={layout} k={k} flags={flags}", flush=True)
    start = inputs.random_lattice(L, L + 7)
    host = start if layout == sd.SD_I8 else inputs.pack_bits(start)
    host = torch.from_numpy(host.reshape(-1).copy()).cuda()
    sigma, tau = sd.new_lattice(L, layout), sd.new_lattice(L, layout)
    flat = [x.reshape(-1).view(host.dtype) for x in (sigma, tau)]
    flat[0].copy_(host)
    obs = torch.full((k // every, 3), -1, dtype=torch.int64, device="cuda")
    sd.sd_run(sigma, tau, L, layout, 0.45, 0.8, SEED, 6, 9, k, obs, every, flags)
    assert sd.sd_debug_last_route() == route
    sig, t, rec = oracle.run(start, 0.45, 0.8, SEED, 6, 9, k, obs_every=every)
    for x, w in zip(flat, (sig, t)):
        have = x.cpu().numpy()
        assert np.array_equal(have.reshape(L, L) if layout == sd.SD_I8 else inputs.unpack_bits(have, L), w)
    assert np.array_equal(obs.cpu().numpy(), rec)


@pytest.mark.parametrize("L,layout", [(512, sd.SD_P64), (640, sd.SD_P64), (1024, sd.SD_I8), (2048, sd.SD_P64)])
def test_tuned_whole_steps_stay_in_bands(tmp_path, L, layout):
    # the grid that the tuner keeps for half-step launches, of either word width,
    # does not take a tuned run off the whole steps, which are twice as quick
    print(f"tuned bands L={L} layout={layout}", flush=True)
    sd.sd_tune(L, layout, str(tmp_path / "tune.json"))
    choice = sd.sd_tuned_choice(L, layout)
    print("tuned", choice, flush=True)
    assert choice[0] == 1
    sigma, tau = sd.new_lattice(L, layout), sd.new_lattice(L, layout)
    sd.sd_init(sigma, L, layout, sd.SD_INIT_UP)
    for run in (sd.sd_run, sd.sd_run_noalloc):
        run(sigma, tau, L, layout, 0.4, 0.6, SEED, 1, 0, 5)
        assert sd.sd_debug_last_route() == sd.SD_ROUTE_BANDS


@pytest.mark.parametrize("L,layout", [(8, sd.SD_P64), (17, sd.SD_I8), (24, sd.SD_P64), (32, sd.SD_P32), (90, sd.SD_I8),
                                      (91, sd.SD_I8), (96, sd.SD_P64), (104, sd.SD_P64), (512, sd.SD_P64),
                                      (544, sd.SD_P32)])
def test_diagonal_correlations_one_or_many_workgroups(oracle, L, layout):
    # sums kept by one workgroup (which overwrites whatever out holds) and split
    # over several, rows of 1 to 256 items, on each side of the division
    print(f"diagonals L={L} layout={layout}", flush=True)
    lat = inputs.random_lattice(L, L + 1)
    host = lat if layout == sd.SD_I8 else inputs.pack_bits(lat)
    dev = torch.from_numpy(host.reshape(-1).copy()).cuda()
    for lmax in sorted({0, 1, L // 2, L - 1}):
        out = torch.full((2, lmax + 1), 12345, dtype=torch.int64, device="cuda")
        sd.sd_corr_diag(dev, L, layout, lmax, out)
        assert np.array_equal(out.cpu().numpy().reshape(-1), oracle.corr_diag(lat, lmax).reshape(-1))


@pytest.mark.parametrize("L,layout", [(78, sd.SD_I8), (79, sd.SD_I8), (72, sd.SD_P64), (80, sd.SD_P64), (255, sd.SD_I8),
                                      (257, sd.SD_I8)])
def test_diagonal_correlations_of_sites(oracle, L, layout):
    # lattices taken site by site, on each side of one workgroup per sum and of
    # a row per workgroup; every shift wraps somewhere
    print(f"diagonals of sites L={L} layout={layout}", flush=True)
    lat = inputs.random_lattice(L, L + 2)
    host = lat if layout == sd.SD_I8 else inputs.pack_bits(lat)
    dev = torch.from_numpy(host.reshape(-1).copy()).cuda()
    for lmax in (1, L - 1):
        out = torch.full((2, lmax + 1), 12345, dtype=torch.int64, device="cuda")
        sd.sd_corr_diag(dev, L, layout, lmax, out)
        assert np.array_equal(out.cpu().numpy().reshape(-1), oracle.corr_diag(lat, lmax).reshape(-1))


@pytest.mark.parametrize("L,layout,n,k", [(384, sd.SD_P64, 1, 3), (448, sd.SD_I8, 7, 20), (512, sd.SD_P64, 1, 30),
                                          (576, sd.SD_I8, 5, 9), (1024, sd.SD_P64, 16, 5), (2112, sd.SD_P64, 1, 12),
                                          (4032, sd.SD_P64, 3, 4), (4096, sd.SD_I8, 1, 6)])
def test_bands_of_uneven_rows(L, layout, n, k):
    # whole steps in bands whose rows the side does not divide evenly, from two
    # rows a band to as many as the LDS holds, rows of 6 to 64 words, shapes
    # that need several bands per CU; against the half-steps of the grid kernels
    print(f"bands L={L} layout={layout} n={n}", flush=True)
    J, q, streams = [0.3 + 0.05 * a for a in range(n)], [0.9] * n, [a + 2 for a in range(n)]
    sig = []
    for a in range(n):
        x = sd.new_lattice(L, layout)
        sd.sd_init(x, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, a)
        sig.append(x)
    tau, first = [torch.zeros_like(x) for x in sig], [x.clone() for x in sig]
    obs = torch.full((n, k, 3), -1, dtype=torch.int64, device="cuda")
    sd.sd_run_many(sig, tau, L, layout, J, q, SEED, streams, 2, k, obs, 1)
    for a in range(n):
        one, two = first[a].clone(), torch.zeros_like(first[a])
        rec = torch.empty((k, 3), dtype=torch.int64, device="cuda")
        sd.sd_run(one, two, L, layout, J[a], q[a], SEED, streams[a], 2, k, rec, 1, sd.SD_FLAG_GLOBAL_KERNELS)
        assert torch.equal(one, sig[a]) and torch.equal(two, tau[a]) and torch.equal(rec, obs[a])
        if a == 0:
            one, two = first[0].clone(), torch.zeros_like(first[0])
            sd.sd_run(one, two, L, layout, J[0], q[0], SEED, streams[0], 2, k, rec, 1)
            assert torch.equal(one, sig[0]) and torch.equal(two, tau[0]) and torch.equal(rec, obs[0])


@pytest.mark.parametrize("L,q", [(8, 0.0), (24, 1.0), (512, 1.0), (720, 0.4), (1024, 1.0), (1456, 1.0)])
def test_replica_tables_and_batches(L, q):
    # 64 replicas against single chains at the sizes where the batch of a
    # wavefront changes (one group, an odd count of groups, 2, 2 with a rest,
    # 8 and 16 groups), with thresholds that all replicas share (q alone sets
    # the classes of unlike neighbours), that share a top byte (strong
    # coupling), and that the largest fields saturate.  Whole numbers: exact.
    print(f"replica tables L={L} q={q}", flush=True)
    J = [1.5 * r / 63 for r in range(62)] + [12.0, -3.0]
    qs = [q] * 64
    rng = np.random.default_rng(L)
    info = np.iinfo(np.int64)
    start = rng.integers(info.min, info.max, size=L * L, dtype=np.int64, endpoint=True)
    sig = torch.from_numpy(start).cuda()
    tau = torch.zeros_like(sig)
    sd.sd_replica_run(sig, tau, L, J, qs, 77, 3, 5, 3)

    def replica(words, r):
        return (2 * ((words.view(np.uint64) >> np.uint64(r)) & np.uint64(1)).astype(np.int8) - 1).reshape(L, L)

    for r in (0, 1, 17, 31, 32, 45, 61, 62, 63):
        s1, t1 = sd.new_lattice(L, sd.SD_P64), sd.new_lattice(L, sd.SD_P64)
        s1.view(torch.uint8).view(-1).copy_(torch.from_numpy(inputs.pack_bits(replica(start, r))))
        sd.sd_run(s1, t1, L, sd.SD_P64, J[r], q, 77, 3, 5, 3, None, 0)
        assert np.array_equal(inputs.unpack_bits(s1.cpu().numpy(), L), replica(sig.cpu().numpy(), r)), r
        assert np.array_equal(inputs.unpack_bits(t1.cpu().numpy(), L), replica(tau.cpu().numpy(), r)), r


@pytest.mark.parametrize("L", [8, 24, 120, 128, 136, 264])
@pytest.mark.parametrize("fill", ["random", "plus", "opposed"])
def test_replica_observables_at_counter_edges(L, fill):
    # less than one site per lane, one workgroup (16384 sites) to the site,
    # one site row more, several; full counters of every quantity.  Whole
    # numbers: exact.
    print(f"replica observables L={L} {fill}", flush=True)
    rng = np.random.default_rng(L)
    info = np.iinfo(np.int64)
    if fill == "random":
        sw, tw = (rng.integers(info.min, info.max, size=L * L, dtype=np.int64, endpoint=True) for _ in range(2))
    else:
        sw = np.full(L * L, -1, dtype=np.int64)
        tw = sw.copy() if fill == "plus" else np.zeros_like(sw)
    out = torch.empty((64, 3), dtype=torch.int64, device="cuda")
    sd.sd_replica_observe(torch.from_numpy(sw).cuda(), torch.from_numpy(tw).cuda(), L, out)
    s, t = (inputs.unpack_replicas(x.view(np.uint64), L).reshape(64, L, L).astype(np.int64) for x in (sw, tw))
    up, right = np.roll(t, -1, axis=1), np.roll(t, -1, axis=2)
    want = np.stack([s.sum((1, 2)), (s * (up + right)).sum((1, 2)), (s * t).sum((1, 2))], axis=1)
    assert np.array_equal(out.cpu().numpy(), want)


@pytest.mark.parametrize("L,n", [(8, 3), (24, 3), (64, 2), (64, 300), (72, 3), (128, 3), (128, 300), (136, 3), (176, 3),
                                 (184, 3), (256, 3), (256, 258), (264, 2)])
def test_recorded_trajectories_by_lanes_per_word(L, n):
    # four, two and one lane per word, partly filled tiles, more chains than
    # CUs, the largest one-word-per-lane lattice and the next size; enough
    # half-steps that some list more sites than the workgroup's list holds.
    # Bits: exact.
    print(f"recorded trajectories L={L} n={n}", flush=True)
    k, W = (60 if n < 10 else 4), L * L // 64
    rng = np.random.default_rng(L + n)
    info = np.iinfo(np.int64)
    starts = torch.from_numpy(rng.integers(info.min, info.max, size=n * W, dtype=np.int64, endpoint=True)).cuda()
    traj = torch.zeros(n * (2 * k + 1) * W, dtype=torch.int64, device="cuda")
    for J, q in ((0.45, 0.7), (1.1, 0.0)):
        sd.sd_trajectories(starts, traj, n, L, sd.SD_P64, J, q, SEED, 7, 3, k)
        for a in {0, 1, n - 1}:
            one = torch.zeros((2 * k + 1) * W, dtype=torch.int64, device="cuda")
            sd.sd_trajectory(starts[a * W:(a + 1) * W].clone(), one, L, sd.SD_P64, J, q, SEED, 7 + a, 3, k)
            assert torch.equal(one, traj.view(n, -1)[a]), (J, q, a)


@pytest.mark.parametrize("L,layout,k", [(64, sd.SD_I8, 100), (100, sd.SD_I8, 40), (256, sd.SD_P64, 40), (200, sd.SD_P64, 40)])
def test_captured_small_run_replayed_beside_its_stream(L, layout, k):
    # a run that is drawn ahead when called eagerly, captured on a stream that
    # has its scratch buffer, then replayed on another stream while eager runs
    # use that buffer: every replay gives the eager run's lattices and records.
    # (The eager runs beside it record nothing: the partial sums of recorded
    # half-step launches are the stream's, in a graph as in a call.)
    print(f"captured small run L={L} layout={layout}", flush=True)
    pair = [[sd.new_lattice(L, layout) for _ in range(2)] for _ in range(2)]
    first = sd.new_lattice(L, layout)
    sd.sd_init(first, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    obs = torch.empty((k, 3), dtype=torch.int64, device="cuda")

    def run(i, stream_id):
        pair[i][0].copy_(first)
        sd.sd_run(pair[i][0], pair[i][1], L, layout, 0.4, 0.6, SEED, stream_id, 0, k, obs if i == 0 else None,
                  1 if i == 0 else 0)

    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        run(0, 5)
    torch.cuda.synchronize()
    want = [t.clone() for t in (*pair[0], obs)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        run(0, 5)
    for _ in range(4):
        for t in (*pair[0], obs):
            t.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(3):
                run(1, 6)
        with torch.cuda.stream(other):
            graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((*pair[0], obs), want))


@pytest.mark.parametrize("L,layout,n,k", [(100, sd.SD_I8, 1, 12), (512, sd.SD_P64, 1, 40), (448, sd.SD_I8, 1, 9),
                                          (6848, sd.SD_P64, 1, 3), (512, sd.SD_P64, 5, 40), (520, sd.SD_P64, 3, 6)])
def test_captured_records_replayed_beside_their_stream(L, layout, n, k):
    # recorded runs of every form that keeps partial sums when called eagerly
    # (one-word tiles, bands, wide tiles; one chain and several), captured on a
    # stream that has its partial-sum buffer and replayed on another while
    # recorded eager runs use that buffer; whole numbers: exact
    print(f"captured records L={L} layout={layout} n={n}", flush=True)
    J, q, ids = [0.3 + 0.05 * a for a in range(n)], [0.8] * n, [a + 2 for a in range(n)]
    first = [sd.new_lattice(L, layout) for _ in range(n)]
    for a in range(n):
        sd.sd_init(first[a], L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, a)
    sets = [[[torch.zeros_like(x) for x in first] for _ in range(2)] for _ in range(2)]
    obs = [torch.full((n, k, 3), -1, dtype=torch.int64, device="cuda") for _ in range(2)]

    def run(i, step0):
        for x, y in zip(sets[i][0], first):
            x.copy_(y)
        if n == 1:
            sd.sd_run(sets[i][0][0], sets[i][1][0], L, layout, J[0], q[0], SEED, ids[0], step0, k, obs[i], 1)
        else:
            sd.sd_run_many(sets[i][0], sets[i][1], L, layout, J, q, SEED, ids, step0, k, obs[i], 1)

    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    want = []
    for step0 in (0, 1000):
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            run(0, step0)
        torch.cuda.synchronize()
        want.append([t.clone() for t in (*sets[0][0], *sets[0][1], obs[0])])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        run(0, 0)
    for _ in range(4):
        for o in obs:
            o.fill_(-1)
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for _ in range(3):
                run(1, 1000)
        with torch.cuda.stream(other):
            graph.replay()
        torch.cuda.synchronize()
        for i in range(2):
            assert all(torch.equal(a, b) for a, b in zip((*sets[i][0], *sets[i][1], obs[i]), want[i])), i


def test_captured_counts_replayed_beside_their_stream():
    # the log-likelihood counts keep partial sums of the same buffer
    n, k, L = 6, 20, 128
    start = torch.empty((n, L * L // 64), dtype=torch.int64, device="cuda")
    for a in range(n):
        sd.sd_init(start[a], L, sd.SD_P64, sd.SD_INIT_RANDOM, 0.5, SEED, a)
    traj = [torch.empty((n, 2 * k + 1, L * L // 64), dtype=torch.int64, device="cuda") for _ in range(2)]
    for i in range(2):
        sd.sd_trajectories(start, traj[i], n, L, sd.SD_P64, 0.4, 0.5 + i, SEED, 0, 0, k)
    out = [torch.zeros(12, dtype=torch.int64, device="cuda") for _ in range(2)]
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for i in range(2):
        sd.sd_loglik_counts(traj[i], n, 2 * k + 1, L, out[i], hip_stream=stream)
    torch.cuda.synchronize()
    want = [o.clone() for o in out]
    assert int(want[0].sum()) == 2 * k * n * L * L
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sd.sd_loglik_counts(traj[0], n, 2 * k + 1, L, out[0])
    for _ in range(4):
        for o in out:
            o.fill_(-1)
        torch.cuda.synchronize()
        for _ in range(3):
            sd.sd_loglik_counts(traj[1], n, 2 * k + 1, L, out[1], hip_stream=stream)
        with torch.cuda.stream(other):
            graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))


@pytest.mark.parametrize("L,layout,k,many", [(64, sd.SD_I8, 60, False), (200, sd.SD_P64, 40, False), (300, sd.SD_I8, 20, False),
                                             (100, sd.SD_I8, 30, True), (512, sd.SD_P64, 30, False), (640, sd.SD_P64, 20, True)])
def test_threads_on_the_per_thread_stream(L, layout, k, many):
    # hipStreamPerThread is one handle, but another queue in every host thread:
    # threads that draw ahead, or keep partial sums of records, on it at the same
    # time get the chains and records that each gets alone
    print(f"per-thread stream L={L} layout={layout} many={many}", flush=True)
    per_thread, n_threads, n_sets = 2, 4, 6   # the handle's value is hipStreamPerThread's
    first = sd.new_lattice(L, layout)
    sd.sd_init(first, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, 1)

    def run(sigma, tau, obs, stream_id, hip_stream=None):
        if many:
            sd.sd_run_many([sigma], [tau], L, layout, [0.4], [0.6], SEED, [stream_id], 0, k, obs, 1, hip_stream=hip_stream)
        else:
            sd.sd_run(sigma, tau, L, layout, 0.4, 0.6, SEED, stream_id, 0, k, obs, 1, hip_stream=hip_stream)

    def sets(n):
        return [(first.clone(), torch.zeros_like(first), torch.full((k, 3), -1, dtype=torch.int64, device="cuda"))
                for _ in range(n)]

    want = sets(n_threads)
    for i, w in enumerate(want):
        run(*w, 10 + i)
    got = [sets(n_sets) for _ in range(n_threads)]
    torch.cuda.synchronize()
    errors, ready = [], threading.Barrier(n_threads)

    def work(i):
        try:
            ready.wait(60)
            for g in got[i]:
                run(*g, 10 + i, hip_stream=per_thread)
            torch.cuda.synchronize()
        except Exception as e:   # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(90)
    assert not errors, errors
    torch.cuda.synchronize()
    for i in range(n_threads):
        for g in got[i]:
            assert all(torch.equal(a, b) for a, b in zip(g, want[i])), i


@pytest.mark.parametrize("L,layout", [(64, sd.SD_I8), (200, sd.SD_P64), (512, sd.SD_P64)])
def test_first_run_on_a_stream_beside_a_capture(L, layout):
    # one thread captures (in the mode that forbids unsafe calls in every
    # thread) while another makes its first runs on a stream, which make the
    # stream's buffers: the capture goes through and the runs are right
    print(f"first run beside a capture L={L} layout={layout}", flush=True)
    k = 40
    first = sd.new_lattice(L, layout)
    sd.sd_init(first, L, layout, sd.SD_INIT_RANDOM, 0.5, SEED, 1)
    sets = [(first.clone(), torch.zeros_like(first), torch.full((k, 3), -1, dtype=torch.int64, device="cuda"))
            for _ in range(2)]
    sd.sd_run(*sets[0][:2], L, layout, 0.4, 0.6, SEED, 1, 0, k, sets[0][2], 1)
    x = torch.zeros(1000, device="cuda")
    capture, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    handle = ctypes.c_void_p()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0   # a handle the library has not seen
    torch.cuda.synchronize()
    errors = []

    def work():
        try:
            sd.sd_run(*sets[1][:2], L, layout, 0.4, 0.6, SEED, 1, 0, k, sets[1][2], 1, hip_stream=handle.value)
        except Exception as e:   # reported by the main thread
            errors.append(e)

    thread = threading.Thread(target=work)
    with torch.cuda.graph(graph, stream=capture):
        x += 1
        thread.start()
        thread.join(60)
        x += 1
    assert not errors, errors
    graph.replay()
    torch.cuda.synchronize()
    assert bool((x == 2).all())
    assert all(torch.equal(a, b) for a, b in zip(*sets))
    assert hip.hipStreamDestroy(handle) == 0


@pytest.mark.parametrize("L,n,rmax", [(64, 1, 0), (64, 16, 63), (448, 3, 200), (448, 1, 447), (1024, 5, 512), (1024, 5, 511),
                                      (1024, 1, 1023), (1024, 16, 64)])
@pytest.mark.parametrize("layout", [sd.SD_I8, sd.SD_P64])
def test_row_correlations_by_chunks_per_workgroup(L, n, rmax, layout):
    # one to sixteen 64-shift chunks per workgroup, the last one partial, rows
    # repeated once in full; exact sums
    print(f"row correlations L={L} n={n} rmax={rmax} layout={layout}", flush=True)
    host = [inputs.random_lattice(L, 50 + a) for a in range(n)]
    lat = []
    for x in host:
        t = sd.new_lattice(L, layout)
        raw = x if layout == sd.SD_I8 else inputs.pack_bits(x)
        t.reshape(-1).view(torch.int8 if layout == sd.SD_I8 else torch.uint8).copy_(torch.from_numpy(raw.reshape(-1).copy()))
        lat.append(t)
    out = torch.full((n, rmax + 1), -1, dtype=torch.int64, device="cuda")
    sd.sd_corr_row_many(lat, L, layout, rmax, out)
    got = out.cpu().numpy()
    for a in range(n):
        x = host[a].reshape(L, L).astype(np.float64)   # circular correlation: whole numbers below 2^53
        f = np.fft.rfft(x, axis=1)
        want = np.rint(np.fft.irfft((f * np.conj(f)).sum(axis=0), n=L)).astype(np.int64)
        assert np.array_equal(got[a], want[:rmax + 1]), a
