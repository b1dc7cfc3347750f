"""Helpers for the GPU parity tests: move a raw trace to the device, run the decoder through the
C ABI binding, bring the statistics block back."""
import numpy as np
import torch

import paper_2505_21661_amd as kp


def geometry(raw: np.ndarray):
    n_wg, W, R, cap, rec_cost, flags = (int(x) for x in raw[2:8])
    return n_wg, W, R, cap, rec_cost, flags


def gpu_decode_bytes(raw: np.ndarray, use_hdr: bool = False, dev_raw=None) -> np.ndarray:
    n_wg, W, R, cap, rec_cost, flags = geometry(raw)
    if dev_raw is None:
        dev_raw = torch.from_numpy(raw.view(np.int32)).cuda()
    out = torch.full((kp.kp_stats_bytes(n_wg, W, R),), 0xAB, dtype=torch.uint8, device="cuda")
    n = n_wg * W * cap
    if use_hdr:
        kp.kp_trace_reduce_hdr(dev_raw, n, kp.make_hdr(n_wg, W, R, cap, rec_cost, flags), out)
    else:
        kp.kp_trace_reduce(dev_raw, n, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def assert_stats_equal(want: np.ndarray, got: np.ndarray, oracle_mod):
    if np.array_equal(want, got):
        return
    a, b = oracle_mod.view_stats(want), kp.parse_stats(got)
    for k in a:
        if isinstance(a[k], int):
            assert a[k] == b[k.replace("waves", "waves_per_wg") if k == "waves" else k], (k, a[k], b.get(k))
    for k in ("hist", "cnt", "sum", "min", "max", "U", "O", "F"):
        assert np.array_equal(a[k], b[k]), (k, a[k], b[k])
    bad = np.argwhere((a["per"]["sum"] != b["per"]["sum"]) | (a["per"]["n"] != b["per"]["n"]) | (a["per"]["max"] != b["per"]["max"]))
    assert bad.size == 0, ("per", bad[:5], a["per"][tuple(bad[0])], b["per"][tuple(bad[0])])
    raise AssertionError("stats blocks differ outside the named fields")


def mostly_sequential_trace(seed, W, R, cap, holes=False):
    """Regions that follow one another, with here and there a region around others, a START without END, an END
    without START and (holes) a record that fails its checks; two workgroups, ragged totals."""
    import inputs

    rng = np.random.default_rng(seed)
    wgs = []
    for _ in range(2):
        evs = []
        for w in range(W):
            t, wave, outer = 0, [], -1
            total = cap + 37 if w == 0 else int(rng.integers(1, cap + cap // 2))
            while len(wave) < total:
                t += int(rng.integers(0, 40))
                r, x = int(rng.integers(0, R)), rng.random()
                if x < 0.01 and outer < 0:
                    outer = r
                    wave.append((inputs.PHASE_START, r, t))
                elif x < 0.02 and outer >= 0:
                    wave.append((inputs.PHASE_END, outer, t))
                    outer = -1
                elif x < 0.025:
                    wave.append((inputs.PHASE_START, r, t))
                elif x < 0.03:
                    wave.append((inputs.PHASE_END, r, t))
                else:
                    wave.append((inputs.PHASE_START, r, t))
                    t += int(rng.integers(0, 900))
                    wave.append((inputs.PHASE_END, r, t))
            evs.append(wave[:total])
        wg = inputs.events_to_wg(evs, cap, flush=False)
        if holes:
            for seg in wg["slots"]:
                for _ in range(len(seg) // 90):
                    i = int(rng.integers(0, len(seg)))
                    seg[i] = (0xFFFFFFFF, seg[i][1])
        wgs.append(wg)
    return inputs.encode_trace(wgs, W, R, cap, rec_cost=7)


def nested_trace(seed, W, R, cap, depth, inner):
    """Regions inside regions: blocks of `depth` STARTs and their ENDs in reverse order, now and then one region
    around `inner` others; two workgroups, wave 0 wrapped."""
    import inputs

    rng = np.random.default_rng(seed)
    wgs = []
    for _ in range(2):
        evs = []
        for w in range(W):
            total, wave, t = (cap + 37 if w == 0 else int(rng.integers(1, cap + 1))), [], 0

            def put(phase, region):
                nonlocal t
                t += int(rng.integers(0, 300))
                wave.append((phase, region, t))

            while len(wave) < total:
                order = [int(x) for x in rng.permutation(R)[:depth]]
                around = int(rng.integers(0, R)) if rng.random() < 0.05 else -1
                if around >= 0:
                    put(inputs.PHASE_START, around)
                for _i in range(inner if around >= 0 else 1):
                    for r in order:
                        put(inputs.PHASE_START, r)
                    for r in reversed(order):
                        put(inputs.PHASE_END, r)
                if around >= 0:
                    put(inputs.PHASE_END, around)
            evs.append(wave[:total])
        wgs.append(inputs.events_to_wg(evs, cap, flush=False))
    return inputs.encode_trace(wgs, W, R, cap, rec_cost=7)


def shared_seq_trace(seed, n_wg, W, R, cap):
    """Workgroups of four kinds in turn: all records in the slots of their seq; some slots swapped; some records that repeat
    the seq of the slot below (one of the two is in its own slot); pairs of records that share a seq outside its slot, which
    holds another one, next to each other and far apart."""
    import inputs

    spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=R, cap_wave=cap, total_per_wave=cap, total_var=cap // 2, seed=seed, p_orphan=0.05)
    raw, _ = inputs.gen_trace(spec)
    raw = raw.copy()
    slots = raw[16 + 32 * n_wg:].reshape(n_wg, W, cap, 2)
    rng = np.random.default_rng(seed)
    for wg in range(n_wg):
        w = int(rng.integers(0, W))
        a = int(rng.integers(0, cap // 4 - 2))
        seg = slots[wg, w]
        if wg % 4 == 1:
            seg[[a, a + 1]] = seg[[a + 1, a]]
        elif wg % 4 == 2:
            seg[a + 1, 0] = (seg[a + 1, 0] & ~np.uint32(0xFFFFF)) | (seg[a, 0] & np.uint32(0xFFFFF))
        elif wg % 4 == 3:
            b = a + (1 if wg % 8 == 3 else cap // 4)
            other, shared = seg[a, 0] & np.uint32(0xFFFFF), seg[b + 1, 0] & np.uint32(0xFFFFF)
            seg[[a, b], 0] = (seg[[a, b], 0] & ~np.uint32(0xFFFFF)) | shared
            seg[b + 1, 0] = (seg[b + 1, 0] & ~np.uint32(0xFFFFF)) | other
    return raw


def damaged_between_clean_trace(seed, n_wg, W, R, cap):
    """Clean and displaced records, and between their workgroups ones with a record that fails its checks, a seq that occurs
    twice, a clock that goes back, a span beyond 32 bits, and without any record."""
    import inputs

    spec = inputs.TraceSpec(n_wg=n_wg, waves=W, n_regions=R, cap_wave=cap, total_per_wave=cap, total_var=cap // 4, seed=seed, dist="lognormal",
                            p0=4.0, p1=1.0, p_orphan=0.02, p_swap=0.002)
    raw, _ = inputs.gen_trace(spec)
    raw = raw.copy()
    heads = raw[16:16 + 32 * n_wg].reshape(n_wg, 32)
    slots = raw[16 + 32 * n_wg:].reshape(n_wg, W, cap, 2)
    rng = np.random.default_rng(seed)
    for wg in range(n_wg):
        seg, a = slots[wg, int(rng.integers(0, W))], int(rng.integers(0, cap // 2))
        if wg % 5 == 1:
            seg[a, 0] |= np.uint32(0x7F000000)
        elif wg % 7 == 2:
            seg[a + 1, 0] = (seg[a + 1, 0] & ~np.uint32(0xFFFFF)) | (seg[a, 0] & np.uint32(0xFFFFF))
        elif wg % 11 == 3:
            heads[wg, 5] += 2
        elif wg % 13 == 4:
            seg[[a, a + 1], 1] = seg[[a + 1, a], 1]
        elif wg % 17 == 5:
            heads[wg, 8:24] = 0
    return raw
