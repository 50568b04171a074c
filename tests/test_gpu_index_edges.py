"""The index builder where its launches change: sequences kept in LDS (512, 4096) or in the workspace, positions per thread of the
map write-out (2^18 tokens), more ends of sequences in a wavefront's positions than it has lanes, empty sequences in front of the
first one, and malformed cu_seqlens in a batch whose first round runs over the chip."""
import ctypes as C
import threading

import numpy as np
import pytest
import torch

from oracle import radix_index
from paper_2601_15013_amd import binding

pytestmark = pytest.mark.gpu


def check(seqs, positions=None):
    lens = [len(s) for s in seqs]
    tok = np.concatenate([np.asarray(s, dtype=np.int32) for s in seqs])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    s_ref, g_ref = radix_index.build_index_trie(tok, cu)
    pos = None
    if positions:
        pos = torch.from_numpy(np.concatenate([np.arange(n) for n in lens]).astype(np.int32) + positions).cuda()
    ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(len(seqs)))
    ws.fill_(0x5A)
    S, G, _, n = binding.radix_build_index(torch.from_numpy(tok).cuda(), pos, torch.from_numpy(cu).cuda(), ws)
    assert n == len(g_ref)
    assert np.array_equal(S.cpu().numpy(), s_ref) and np.array_equal(G[:n].cpu().numpy(), g_ref)


def batch(rng, B, lo, hi, alphabet=3, empty=0.0):
    """Sequences over a tiny alphabet: they branch at every level, and many are equal."""
    return [rng.integers(0, alphabet, 0 if rng.random() < empty else rng.integers(lo, hi + 1)) for _ in range(B)]


@pytest.mark.parametrize("B", [511, 512, 513, 1024, 1025, 4095, 4096, 4097])
@pytest.mark.parametrize("positions", [0, 7])
def test_around_the_state_kept_in_lds(B, positions):
    check(batch(np.random.default_rng(B), B, 1, 9, empty=0.1), positions)


@pytest.mark.parametrize("extra", [-1, 0, 1, 255, 1025])
def test_around_the_positions_of_a_thread(extra):
    rng = np.random.default_rng(extra + 5)
    n = (1 << 18) + extra
    prefix = rng.integers(0, 50, 300)
    seqs, left = [], n
    while left > 0:
        k = min(left, int(rng.integers(301, 700)))
        seqs.append(np.concatenate([prefix, rng.integers(0, 50, 400)])[:k])
        left -= k
    check(seqs)


def test_many_ends_within_a_wavefronts_positions():
    rng = np.random.default_rng(9)
    short = batch(rng, 3000, 1, 2, alphabet=40)                       # 64 ends and more within 64 positions and within 256
    check(short[:150])
    long = [rng.integers(0, 40, 1 << 17) for _ in range(2)]
    check(long[:1] + short + long[1:] + short[::-1])


@pytest.mark.parametrize("lead", [1, 63, 64, 65, 130])
def test_empty_sequences_in_front(lead):
    rng = np.random.default_rng(lead)
    check([rng.integers(0, 3, 0)] * lead + batch(rng, 200, 40, 90, alphabet=2, empty=0.2))


@pytest.mark.parametrize("lead", [63, 64, 4000, 4200, 70000])
def test_long_runs_of_empty_sequences(lead):
    rng = np.random.default_rng(lead)
    own = batch(rng, 130, 40, 90, alphabet=2)
    none = [rng.integers(0, 3, 0)]
    check(none * lead + own[:70] + none * 65 + own[70:])


def test_empty_sequences_in_front_cost_no_more_than_behind():
    # every wavefront of the first round looks for the first sequence with tokens
    k, B = 200, 400000
    seqs = [np.concatenate([np.arange(20), [i], np.arange(10)]) for i in range(k)]
    tok = torch.from_numpy(np.concatenate(seqs).astype(np.int32)).cuda()
    ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(B))
    took = {}
    for kind, lens in (("front", [0] * (B - k) + [31] * k), ("behind", [31] * k + [0] * (B - k))):
        cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            binding.radix_build_index(tok, None, cu, ws)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        took[kind] = min(times)
    assert took["front"] < 3 * took["behind"], took        # walked to, 999 800 of them took 145 times as long


@pytest.mark.parametrize("B", [300, 5000])
@pytest.mark.parametrize("fault", ["falls", "past the end", "negative", "starts late", "ends early"])
def test_malformed_ends_in_a_batch_over_the_chip(fault, B):
    n = 100
    cu = np.arange(B + 1, dtype=np.int32) * n
    if fault == "falls":
        cu[150] = cu[149] - 40
    elif fault == "past the end":
        cu[150:299] = B * n + 1000
    elif fault == "negative":
        cu[1] = -5
    elif fault == "starts late":
        cu[0] = 3
    else:
        cu[B] = B * n - 1
    tok = torch.zeros(B * n, dtype=torch.int32, device="cuda")
    ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(B))
    S, G = (torch.full((B * n,), -7, dtype=torch.int32, device="cuda") for _ in range(2))
    with pytest.raises(binding.RadixError) as e:
        binding.radix_build_index(tok, None, torch.from_numpy(cu).cuda(), ws, S, G)
    assert e.value.code == -6
    assert bool((S == -7).all()) and bool((G == -7).all()), "the maps were written"


def test_threads_and_streams_get_their_own_answers():
    # N' and the status come back through pinned host memory that calls share
    wrong = []

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            n = 50 + 13 * i
            tok = torch.arange(2 * n, dtype=torch.int32, device="cuda") % n                 # two equal sequences of n tokens
            cu = torch.tensor([0, n, 2 * n], dtype=torch.int32, device="cuda")
            bad = tok.clone()
            bad[n + 3] = -1
            ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(2))
            for _ in range(50):
                if binding.radix_build_index(tok, None, cu, ws, stream=stream)[3] != n:
                    wrong.append(i)
                try:
                    binding.radix_build_index(bad, None, cu, ws, stream=stream)
                    wrong.append(-i)
                except binding.RadixError as e:
                    if e.code != -7:
                        wrong.append(e.code)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_calls_that_fail_inside_a_capture_keep_no_words():
    lib = binding.load_library()
    n = 300
    tok = torch.arange(2 * n, dtype=torch.int32, device="cuda") % n
    cu = torch.tensor([0, n, 2 * n], dtype=torch.int32, device="cuda")
    ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(2))
    S, G, n_dev, _ = binding.radix_build_index(tok, None, cu, ws)
    torch.cuda.synchronize()
    assert lib.radix_debug_index_host_slots() == 64
    n_host = C.c_int32(-1)
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    for _ in range(3):
        stream, graph = C.c_void_p(), C.c_void_p()
        assert lib.hipStreamCreate(C.byref(stream)) == 0
        assert lib.hipStreamBeginCapture(stream, 2) == 0                # relaxed
        rc = lib.radix_build_index(p(tok), None, p(cu), 2, 2 * n, p(S), p(G), p(n_dev), C.byref(n_host), p(ws), ws.numel(), stream)
        lib.hipStreamEndCapture(stream, C.byref(graph))                 # the wait has ended it: no graph
        lib.hipGetLastError()
        assert rc < 0 and n_host.value == -1
    assert lib.radix_debug_index_host_slots() == 64
    assert binding.radix_build_index(tok, None, cu, ws)[3] == n


def test_a_batch_near_the_largest_number_of_tokens():
    N = 2 ** 31 - 600
    tok = torch.zeros(N, dtype=torch.int32, device="cuda")
    cu = torch.tensor([0, N], dtype=torch.int32, device="cuda")
    ws = binding.alloc_workspace(binding.radix_index_workspace_bytes(1))
    S, G, _, n = binding.radix_build_index(tok, None, cu, ws)
    assert n == N
    for a in range(0, N, 1 << 28):
        want = torch.arange(a, min(N, a + (1 << 28)), dtype=torch.int32, device="cuda")
        assert torch.equal(S[a:a + (1 << 28)], want) and torch.equal(G[a:a + (1 << 28)], want), a
