"""pcm_score_phases on each of its routes, at the sizes where one takes over from another: one workgroup for the smallest batches, a
table per trajectory or slice for ordinary ones, accumulators beyond.  Bit-exact against the CPU checker (integer sums)."""
import numpy as np
import pytest
import torch

from oracle import pcm_oracle as O

pytestmark = pytest.mark.gpu


def batch(n_groups, G, N, A, K, seed, ragged=True):
    rng = np.random.default_rng(seed)
    T = n_groups * G
    reward = (rng.random(T) < 0.5).astype(np.uint8)
    if n_groups > 1:
        reward[:G] = 1                                       # one group without a score
    phase = rng.integers(0, K + 1, size=(T, N)).astype(np.uint8)   # ids beyond the last phase count as the last
    phase[T // 2:] = np.sort(phase[T // 2:], axis=1)
    n_chunks = rng.integers(0, N + 1, size=T).astype(np.int32) if ragged else np.full(T, N, np.int32)
    n_chunks[-1] = N + 3                                     # beyond the slots: clamped
    actions = rng.uniform(-1.0, 1.0, size=(T, N, A)).astype(np.float32)
    return actions, phase, reward, n_chunks


@pytest.mark.parametrize("n_groups,G,N,A,K", [
    (1, 2, 1, 1, 1),            # the least there is
    (2, 8, 36, 56, 4),          # 576 chunks, 8 for each of the 73 threads of a vector: the most that one workgroup takes
    (2, 8, 37, 56, 4),          # one slot more: tables
    (1, 64, 9, 56, 12),         # a group as wide as a wavefront, one workgroup
    (1, 64, 10, 56, 12),        # the same with tables
    (1, 65, 10, 56, 12),        # and wider than one: accumulators
    (40, 2, 7, 56, 2),          # more pair terms than one workgroup forms
    (1, 8, 256, 56, 12),        # few trajectories of one go: accumulators
    (1, 8, 300, 56, 12),        # five slices of a trajectory
    (1, 2, 700, 4, 3),          # slices of unequal length; one vector per chunk
    (3, 5, 50, 7, 9),           # single floats
    (2, 4, 16, 256, 31),        # pair terms of eight workgroups; almost all of LDS for the sums of a trajectory
    (2, 4, 16, 256, 32),        # more than LDS holds: accumulators
    (2, 4, 30, 256, 31),        # eight trajectories in one go: accumulators
    (64, 8, 20, 56, 18),        # 4.0 MB of tables
    (64, 8, 20, 56, 19),        # and 4.2: accumulators
    (90, 3, 5, 3, 64),          # pair scores of several rounds through LDS in the mean
    (4, 32, 40, 200, 9),        # five threads a sum for 64 tables, a phase per workgroup
    (11, 9, 20, 75, 5),         # three threads a sum for 18 tables
    (8, 8, 73, 56, 5),          # narrow workgroups for the slices: 1022 vectors (wide ones for single floats)
    (2, 8, 128, 32, 8),         # 1024 vectors, and as many sums as narrow workgroups form
    (13, 8, 129, 32, 9),        # one slot more in two slices, more sums
    (3, 4, 60, 68, 3),          # 1020 vectors
    (25, 4, 61, 68, 3),         # 1037 in slices of 31 slots
    (2, 2, 4, 256, 31),         # wide workgroups for the sums, narrow ones for the slices
    (8, 64, 3, 8, 3),           # 512 trajectories
    (27, 19, 3, 8, 3),          # and 513
    (12, 64, 3, 8, 3),          # 768
    (70, 11, 3, 8, 3),          # and 770: accumulators
    (20, 8, 292, 56, 5),        # four slices, each in one go
    (20, 8, 293, 56, 5),        # one slot more than one go: accumulators
    (16, 8, 320, 255, 2),       # four slices of 20 chunks a thread
    (16, 8, 324, 255, 2),       # and of 21: accumulators
    (43, 3, 40, 255, 2),        # more than four chunks a thread and 129 trajectories: accumulators
    (12, 8, 128, 56, 5),        # 96 trajectories in one go: accumulators
    (97, 1, 128, 56, 5),        # and 97: several slices
    (128, 4, 6, 5, 3),          # as many groups as tables take
    (129, 3, 6, 5, 3),          # and one more: accumulators
])
@pytest.mark.parametrize("largest", [1.0, 2.0 ** 20])       # the limit of the definition: sums of whole numbers up to 2^44
def test_score_routes(n_groups, G, N, A, K, largest):
    import paper_2605_16154_amd as pcm
    actions, phase, reward, n_chunks = batch(n_groups, G, N, A, K, seed=N + K)
    actions = np.clip(actions * np.float32(1.5 * largest), -largest, largest)
    dev = lambda x: torch.from_numpy(x).cuda()
    for counts in (n_chunks, None):
        C_o, valid_o = O.phase_scores(actions, phase, reward, None if counts is None else np.minimum(counts, N), n_groups, G, K)
        adv_o, active_o = O.advantages(reward, G)
        shifted = torch.empty(actions.size + 1, device="cuda")[1:].view(actions.shape)      # not aligned to a vector
        shifted.copy_(dev(actions))
        for acts in (dev(actions), shifted):
            out = (torch.full((K,), 7.0, dtype=torch.float64, device="cuda"), torch.full((K,), 9, dtype=torch.uint8, device="cuda"),
                   torch.full((n_groups * G,), 7.0, device="cuda"), torch.full((n_groups * G,), 9, dtype=torch.uint8, device="cuda"))
            for _ in range(2):                               # the second time on scratch that the first has used
                C, valid, adv, active = pcm.pcm_score_phases(acts, dev(phase), dev(reward), None if counts is None else dev(counts), n_groups, G,
                                                             K, 1e-6, out=out)
                assert np.array_equal(C.cpu().numpy().view(np.int64), C_o.view(np.int64))
                assert np.array_equal(valid.cpu().numpy(), valid_o)
                assert np.array_equal(active.cpu().numpy(), active_o)
                assert np.allclose(adv.cpu().numpy(), adv_o, rtol=1e-6, atol=0)


@pytest.mark.parametrize("shape", [(2, 8, 32, 56, 4), (32, 8, 64, 56, 5), (2, 4, 30, 256, 32)])
def test_the_accumulators_bound_the_workspace_on_every_route(shape):
    """Less than the accumulators is refused, and they are enough, also where the query asks for more."""
    import paper_2605_16154_amd as pcm
    L = pcm.lib()
    n_groups, G, N, A, K = shape
    actions, phase, reward, n_chunks = batch(*shape, seed=3)
    C_o, valid_o = O.phase_scores(actions, phase, reward, np.minimum(n_chunks, N), n_groups, G, K)
    a, ph, r, nc = (torch.from_numpy(x).cuda() for x in (actions, phase, reward, n_chunks))
    C, valid = torch.zeros(K, dtype=torch.float64, device="cuda"), torch.zeros(K, dtype=torch.uint8, device="cuda")
    accumulators = n_groups * K * (2 * A * 8 + 2 * 4 + 8 + 1)
    enough = accumulators + 4 * 256                          # four arrays, each from a multiple of 256 bytes on
    ws = torch.zeros(enough, dtype=torch.uint8, device="cuda")
    args = (a.data_ptr(), ph.data_ptr(), r.data_ptr(), nc.data_ptr(), *shape, 1e-6, C.data_ptr(), valid.data_ptr(), None, None)
    stream = torch.cuda.current_stream().cuda_stream
    assert L.pcm_score_phases_workspace_bytes(*shape) >= accumulators
    for p, size in ((None, 0), (ws.data_ptr(), accumulators - 1)):
        assert L.pcm_score_phases(*args, p, size, stream) == -2
    assert L.pcm_score_phases(*args, ws.data_ptr(), enough, stream) == 0
    assert np.array_equal(C.cpu().numpy().view(np.int64), C_o.view(np.int64))
    assert np.array_equal(valid.cpu().numpy(), valid_o)


@pytest.mark.parametrize("n_groups,G,N,A,K", [(2, 8, 32, 56, 4), (3, 5, 12, 7, 3), (32, 8, 64, 56, 5), (3, 5, 50, 7, 9), (2, 4, 30, 256, 32)])
def test_values_beyond_the_required_range(n_groups, G, N, A, K):
    """|a| <= 2^20 is what the definition asks for.  Larger values still add up exactly, as integers, whichever route a batch takes, and
    a NaN counts as 0 without touching the values around it."""
    import paper_2605_16154_amd as pcm
    actions, phase, reward, n_chunks = batch(n_groups, G, N, A, K, seed=N)
    dev = lambda x: torch.from_numpy(x).cuda()
    score = lambda a: [t.cpu().numpy() for t in pcm.pcm_score_phases(dev(a), dev(phase), dev(reward), dev(n_chunks), n_groups, G, K, 1e-6)[:2]]
    where = np.random.default_rng(K).random(actions.shape)
    large = np.where(where < 0.05, actions * np.float32(2.0 ** 30), actions).astype(np.float32)      # sums below 2^63
    C, valid = score(large)
    C_o, valid_o = O.phase_scores(large, phase, reward, np.minimum(n_chunks, N), n_groups, G, K)
    assert np.array_equal(C.view(np.int64), C_o.view(np.int64)) and np.array_equal(valid, valid_o)
    C, valid = score(np.where(where < 0.02, np.float32(np.nan), actions))
    C_0, valid_0 = score(np.where(where < 0.02, np.float32(0.0), actions))
    assert np.array_equal(C.view(np.int64), C_0.view(np.int64)) and np.array_equal(valid, valid_0)
