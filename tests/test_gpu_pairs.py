"""GPU parity of kp_trace_pairs (timeline rows) against oracle/ref_pairs.c, through the C ABI.

Bit-exact: counts, the first count rows of every (workgroup, wave), and the untouched remainder.
"""
import json
import math

import numpy as np
import pytest

import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kp():
    import paper_2505_21661_amd as kp

    return kp


def run_pairs(kp, raw, use_hdr=False, fill=0xA5):
    n_wg, W, R, cap = (int(x) for x in raw[2:6])
    n = n_wg * W * cap
    dev = torch.from_numpy(raw.view(np.int32)).cuda()
    out = torch.full((max(16, kp.kp_pairs_bytes(n_wg, W, W * cap)),), fill, dtype=torch.uint8, device="cuda")
    if use_hdr:
        kp.kp_trace_pairs_hdr(dev, n, kp.make_hdr(n_wg, W, R, cap, int(raw[6]), int(raw[7])), out)
    else:
        kp.kp_trace_pairs(dev, n, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()[: kp.kp_pairs_bytes(n_wg, W, W * cap)]


def assert_pairs_equal(oracle_mod, raw, got, fill=0xA5):
    ref = oracle_mod.pairs_raw(raw, fill=fill)
    assert got.size == ref.size
    if not np.array_equal(ref, got):
        n_wg, W, _R, cap = (int(x) for x in raw[2:6])
        rc, rr = oracle_mod.view_pairs(ref, n_wg, W, cap)
        gc, gr = oracle_mod.view_pairs(got, n_wg, W, cap)
        assert np.array_equal(rc, gc), ("count", np.argwhere(rc != gc)[:5])
        bad = np.argwhere(rr != gr)
        raise AssertionError(f"rows differ at {bad[:5].tolist()}: ref {rr[tuple(bad[0])]} got {gr[tuple(bad[0])]}")


@pytest.mark.parametrize("seed", range(12))
def test_messy_traces(kp, oracle_mod, seed):
    waves = [1, 2, 3, 4, 5, 8, 16][seed % 7]
    n_regions = [1, 3, 5, 16, 17, 32, 100][seed % 7]
    cap = [2, 8, 32, 64, 128, 256][seed % 6]
    raw = inputs.messy_trace(2000 + seed, n_wg=9, waves=waves, n_regions=n_regions, cap_wave=cap,
                             flush=bool(seed & 1))
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw, use_hdr=bool(seed & 2)))


@pytest.mark.parametrize("W,R,cap,total", [(4, 3, 128, 48), (8, 16, 2048, 2048), (8, 16, 2048, 6144),
                                           (4, 7, 4096, 4096), (1, 2, 16384, 16384), (16, 16, 1024, 1000),
                                           (4, 128, 1024, 1024), (2, 100, 512, 700), (3, 65, 256, 256)])
def test_generated_traces(kp, oracle_mod, W, R, cap, total):
    spec = inputs.TraceSpec(n_wg=37, waves=W, n_regions=R, cap_wave=cap, total_per_wave=total, total_var=total // 3,
                            seed=W * 1000 + R, p_orphan=0.02, p_swap=1e-3)
    raw, _ = inputs.gen_trace(spec)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw))


@pytest.mark.parametrize("W,R,cap,depth,inner", [(1, 128, 4096, 2, 3), (4, 5, 1024, 3, 40), (8, 16, 2048, 6, 12), (3, 32, 128, 17, 2), (16, 2, 64, 2, 9)])
def test_regions_inside_regions(kp, oracle_mod, W, R, cap, depth, inner):
    """ENDs whose START lies up to some hundreds of records back, two of them next to each other among them."""
    from tests.gpu_util import nested_trace

    raw = nested_trace(R + depth, W, R, cap, depth, inner)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw))


@pytest.mark.parametrize("holes", [False, True])
@pytest.mark.parametrize("W,R,cap", [(1, 128, 2048), (3, 7, 1024), (16, 16, 256), (8, 33, 128), (5, 3, 64), (2, 5, 8192)])
def test_mostly_sequential_traces(kp, oracle_mod, W, R, cap, holes):
    """Rounds of two ranks per lane next to rounds that have to look further back, in runs of every length."""
    from tests.gpu_util import mostly_sequential_trace

    raw = mostly_sequential_trace(17 * W + R, W, R, cap, holes)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw, use_hdr=True))


@pytest.mark.parametrize("W,cap", [(1, 512), (1, 1024), (1, 2048), (3, 2048), (5, 512), (2, 8192), (1, 16384)])
def test_runs_of_a_wave_that_is_cut_up(kp, oracle_mod, W, cap):
    """Three and more parts per recorded wave (two for 5 waves of 512): record counts around the rounds of 128 that the
    parts are made of, a region that is open across the cuts, pairs whose records lie on either side of one, and
    records that fail their checks right below a cut."""
    rng = np.random.default_rng(W + cap)
    wgs = []
    for total in (0, 1, 2, 127, 128, 129, 255, 257, cap // 2 - 1, cap - 128, cap - 1, cap, cap + 1, cap + 129):
        evs = []
        for w in range(W):
            n = max(0, total - 3 * w)
            wave = [(inputs.PHASE_START, 6, 1)] if w != 1 else []
            while len(wave) < n - 1:
                t = 10 * len(wave)
                r = int(rng.integers(0, 6))
                wave += [(inputs.PHASE_START, r, t), (inputs.PHASE_END, r, t + int(rng.integers(0, 12)))]
            wave = wave[:max(0, n - 1)] + [(inputs.PHASE_END, 6, 10 * n + 20)] * (n > 0)
            evs.append(wave)
        wg = inputs.events_to_wg(evs, cap, flush=False)
        if total % 2:
            for seg in wg["slots"]:
                for i in range(127, len(seg), 256):
                    seg[i] = (0xFFFFFFFF, seg[i][1])
        wgs.append(wg)
    raw = inputs.encode_trace(wgs, W, 7, cap, rec_cost=3)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw, use_hdr=True))


@pytest.mark.parametrize("W,cap", [(1, 512), (1, 1024), (3, 2048), (2, 8192), (1, 16384)])
def test_first_record_of_a_wave_that_is_cut_up(kp, oracle_mod, W, cap):
    """A wave that begins with an END has nothing below that record, whatever its runs end in: here each ends in a
    START of the same region."""
    wgs = []
    for total in (1, 127, 128, 129, 256, 384, cap // 2, cap - 2, cap, cap + 2):
        wave = [(inputs.PHASE_START if k % 2 else inputs.PHASE_END, 0, 10 * k) for k in range(total)]
        wgs.append(inputs.events_to_wg([wave] * W, cap, flush=False))
    raw = inputs.encode_trace(wgs, W, 1, cap, rec_cost=3)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw, use_hdr=True))


# rings of 64 (a hardware wave's 128 records are several recorded waves') and of 128 and more; several turns each
@pytest.mark.parametrize("n_wg,W,R,cap", [(3001, 3, 5, 64), (3002, 3, 5, 128), (1205, 5, 16, 512), (603, 8, 7, 1024)])
def test_shared_seq_in_every_other_turn(kp, oracle_mod, n_wg, W, R, cap):
    from tests.gpu_util import shared_seq_trace

    raw = shared_seq_trace(n_wg, n_wg, W, R, cap)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw, use_hdr=True))


def test_many_workgroups_exercise_generation_reuse(kp, oracle_mod):
    # more recorded workgroups than resident decoder workgroups: the staging area is reused
    spec = inputs.TraceSpec(n_wg=3000, waves=4, n_regions=6, cap_wave=64, total_per_wave=64, total_var=40, seed=77,
                            p_orphan=0.05, p_swap=0.01)
    raw, _ = inputs.gen_trace(spec)
    assert_pairs_equal(oracle_mod, raw, run_pairs(kp, raw, use_hdr=True))


def test_single_region_many_pairs_per_round(kp, oracle_mod):
    # one region: 32 pairs in every round of 64 ranks, the largest per-round counter value
    ev = []
    for i in range(256):
        ev += [(inputs.PHASE_START, 0, 10 * i), (inputs.PHASE_END, 0, 10 * i + 7)]
    wg = inputs.events_to_wg([ev, ev[:100]], 512)
    raw = inputs.encode_trace([wg], 2, 1, 512)
    got = run_pairs(kp, raw)
    assert_pairs_equal(oracle_mod, raw, got)
    count, rows = kp.parse_pairs(got, 1, 2, 1024)
    assert count.tolist() == [[256, 50]] and rows[0, 0, :256]["iter"].tolist() == list(range(256))


def test_empty_and_argument_errors(kp):
    raw = inputs.encode_trace([], 2, 3, 8)
    dev = torch.from_numpy(raw.view(np.int32)).cuda()
    out = torch.zeros(16, dtype=torch.uint8, device="cuda")
    kp.kp_trace_pairs(dev, 0, out)
    with pytest.raises(kp.KperfError):
        kp.kp_trace_pairs(dev, 5, out)  # slot count does not match the header


def test_rows_of_a_real_gemm_trace_and_chrome_export(kp, oracle_mod, tmp_path):
    from paper_2505_21661_amd import timeline

    M = N = 1024
    K = 512
    a, b = inputs.gemm_inputs(M, N, K, seed=5)
    A, B = a.cuda(), b.cuda()
    C = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    n_wg, waves, R = kp.kp_gemm_launch_shape(M, N, K)
    cap = 1024
    trace = torch.zeros(kp.kp_trace_bytes(n_wg, waves, cap), dtype=torch.uint8, device="cuda")
    kp.kp_gemm_instrumented(A, B, C, M, N, K, (1 << R) - 1, trace, cap)
    out = torch.zeros(kp.kp_pairs_bytes(n_wg, waves, cap), dtype=torch.uint8, device="cuda")
    kp.kp_trace_pairs(trace, n_wg * cap, out)
    torch.cuda.synchronize()
    raw = trace.cpu().numpy().view(np.uint32).copy()
    got = out.cpu().numpy()
    assert_pairs_equal(oracle_mod, raw, got, fill=0)
    count, rows = kp.parse_pairs(got, n_wg, waves, cap)
    kt = K // 64
    assert (count == 3 * kt + 1).all()
    r0 = rows[3, 5, : count[3, 5]]
    # per K step: first half, second half, barrier wait; then the epilogue once
    assert r0["region"].tolist() == [0, 1, 2] * kt + [3]
    assert r0["iter"].tolist() == [i for i in range(kt) for _ in range(3)] + [0]
    assert (np.diff(r0["start"].astype(np.int64)) > 0).all()
    path = tmp_path / "gemm_trace.json"
    n_ev = timeline.write_chrome_trace(str(path), count, rows, ["mfma+A", "mfma+B", "barrier", "epilogue"],
                                       ticks_per_us=2300.0, max_wgs=2)
    doc = json.loads(path.read_text())
    assert n_ev == len(doc["traceEvents"]) == 2 * waves * (3 * kt + 1)
    ev = doc["traceEvents"][0]
    assert ev["ph"] == "X" and ev["name"] == "mfma+A" and ev["args"]["iter"] == 0 and ev["dur"] > 0
