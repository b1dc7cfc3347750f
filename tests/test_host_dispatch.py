"""Which kernels a call launches, and which geometries it takes, on devices of several sizes (no GPU needed)."""
import pytest

from tests import fake_hip


def kernels(launches, part):
    return [x for x in launches if part in x[0]]


def test_statistics_are_derived_exactly_once(tmp_path):
    """The figures are derived behind the main kernel, once, also where a small device (a partition of the chip) holds
    fewer decoder workgroups than the trace has."""
    calls = []
    for dev, (cus, per_cu) in enumerate([(256, 2), (64, 2), (32, 2), (32, 3), (20, 1), (32, 8)]):
        for waves, regions, cap in ((4, 3, 128), (8, 5, 512), (8, 16, 2048), (8, 40, 64)):
            for n_wg in (1, 127, 128, 129, 200, 1000):
                calls.append({"fn": "kp_trace_reduce_hdr", "trace": (n_wg, waves, regions, cap), "device": (dev, cus, per_cu)})
    for call, (status, launches) in zip(calls, fake_hip.run(calls, tmp_path)):
        assert status == 0, call
        n_wg, (_, cus, per_cu) = call["trace"][0], call["device"]
        main, derive = launches[1:-1], launches[-1]
        assert len(main) == 1 and main[0][1] == min(n_wg, cus * per_cu), (call, launches)
        assert "kp_reduce_derive" in derive[0] and derive[1:3] == (1, 1024), (call, launches)


# (waves, cap_wave, regions): the most regions whose sums fit the LDS beside the staged records, one copy of the sums
WAITS_LIMITS = [(1, 16384, 100), (2, 8192, 95), (4, 4096, 87), (7, 2048, 116), (8, 2048, 74), (13, 1024, 110),
                (14, 1024, 92), (15, 1024, 74), (16, 1024, 57)]


def test_wait_replay_takes_every_geometry_up_to_its_limit(tmp_path):
    shapes = [(w, r, cap) for w, cap, r0 in WAITS_LIMITS for r in (1, r0 - 1, r0, r0 + 1)]
    calls = [{"fn": "kp_trace_waits_hdr", "trace": (3, *s)} for s in shapes]
    limit = {(w, cap): r0 for w, cap, r0 in WAITS_LIMITS}
    for (w, r, cap), (status, launches) in zip(shapes, fake_hip.run(calls, tmp_path)):
        assert (status == 0) == (r <= limit[w, cap]), (w, r, cap, status)
        assert all(lds <= 160 * 1024 for _, _, _, lds in launches), launches


def test_wait_header_counts_are_made_once(tmp_path):
    """The three header counts are added by the decoder workgroups or made by a kernel behind them: the line goes by
    the launched grid, also where a small device holds fewer workgroups than the trace has."""
    calls = [{"fn": "kp_trace_waits_hdr", "trace": (n_wg, 8, regions, 64), "device": (dev, cus, 2)}
             for dev, cus in enumerate((256, 64, 8)) for regions in (1, 4, 6, 7, 16, 21, 57) for n_wg in (1, 74, 75, 219, 224, 5000)]
    for call, (status, launches) in zip(calls, fake_hip.run(calls, tmp_path)):
        assert status == 0, call
        n_wg, _, regions, _ = call["trace"]
        each = max(1, int((n_wg / (64 + 8 * 64 / 48)) ** 0.5 + 0.5))
        grid = min(2 * call["device"][1], -(-n_wg // each))
        main = kernels(launches, "kp_waits_main")
        assert len(main) == 1 and main[0][1] == grid, (call, launches)
        head = kernels(launches, "kp_waits_head")
        added = regions <= 20 and (grid <= 128 or regions in (1, 6, 7))
        assert [x[1:3] for x in head] == ([] if added else [(1, 192)]), (call, launches)
        assert not head or launches[-1] == head[0]


def test_wait_header_counts_of_odd_region_counts(tmp_path):
    """With more than nine regions the totals of a decoder workgroup take two hardware waves: many workgroups leave the header
    counts to the kernel behind them, few add them all the same."""
    calls = [{"fn": "kp_trace_waits_hdr", "trace": (n_wg, 4, regions, 256), "device": (0, 256, 2)} for regions in (9, 11, 19) for n_wg in (100, 3000)]
    for call, (status, launches) in zip(calls, fake_hip.run(calls, tmp_path)):
        n_wg, _, regions, _ = call["trace"]
        assert status == 0 and (len(kernels(launches, "kp_waits_head")) == 0) == (n_wg == 100 or regions == 9), (call, launches)


@pytest.mark.parametrize("tiles,k_max", [((17, 15), 0), ((257, 1), 96), ((256, 3), 96), ((769, 1), 160), ((33, 31), 160), ((41, 25), 224), ((3071, 1), 224), ((63, 62), 288)])
def test_short_k_gemm_has_one_line_for_every_way_of_recording(tmp_path, tiles, k_max):
    """Which 64x64x32 kernel a shape takes does not depend on what is recorded, so that a recorded kernel and the one
    without sites are the same; circular records of one lane keep the chained sites in both."""
    kernel = {0: 0, 7: 2, 5: 2, 7 | 1 << 30: 2, 7 | 1 << 28: 5, 7 | 1 << 31: 1, 7 | 1 << 27: 1, 7 | 1 << 27 | 1 << 28: 3}
    calls = [{"fn": "kp_gemm_instrumented", "args": (64 * tiles[0], 64 * tiles[1], k, mask, 256)}
             for k in (32, 96, 128, 160, 192, 224, 256, 288, 320, 4128) for mask in kernel]
    for call, (status, launches) in zip(calls, fake_hip.run(calls, tmp_path)):
        assert status == 0, call
        k, mask = call["args"][2:4]
        name = "kp_gemm_short" if k <= k_max else "kp_gemm_small"
        assert len(launches) == 1 and f"{name}ILi{kernel[mask]}E" in launches[0][0], (call, launches)
        assert launches[0][1] == tiles[0] * tiles[1]


@pytest.mark.parametrize("device", [(0, 256, 8), (1, 256, 6), (2, 32, 8)])
def test_critical_path_workgroups_are_bounded_by_their_totals(tmp_path, device):
    """Never more decoder workgroups than recorded ones or than seven per CU, all of them where few are recorded, and
    otherwise a number near the root of the recorded ones that gives each as many of them as the others."""
    shapes = [(n_wg, r, i) for n_wg in (1, 2, 450, 513, 1024, 1025, 2048, 5000, 65536) for r, i in ((1, 1), (1, 64), (5, 13), (16, 64), (128, 32))]
    calls = [{"fn": "kp_stages_critical", "args": s, "device": device} for s in shapes]
    for (n_wg, r, i), (status, launches) in zip(shapes, fake_hip.run(calls, tmp_path)):
        assert status == 0 and "kp_critical_main" in launches[-1][0], (n_wg, r, i, launches)
        places = 64
        while places < r * i:
            places *= 2
        grid, resident = launches[-1][1], min(7, device[2]) * device[1]
        root = (n_wg * (450 + places)) ** 0.5
        assert 1 <= grid <= min(n_wg, resident)
        assert grid == min(n_wg, resident) or (n_wg > 450 + places and root / 2 <= grid <= 2 * root)
        turns = -(-n_wg // grid)
        assert grid == resident or grid == -(-n_wg // turns)


@pytest.mark.parametrize("device", [(0, 256, 8), (1, 256, 4), (2, 32, 8)])
def test_timeline_workgroups_of_small_rings(tmp_path, device):
    """Blocks of 256 threads: at most six per CU; larger ones as many as are resident."""
    shapes = [(n_wg, w, cap) for n_wg in (1, 191, 193, 1537, 40000) for w, cap in ((1, 256), (4, 256), (2, 32), (8, 64), (8, 2048))]
    calls = [{"fn": "kp_trace_pairs_hdr", "trace": (n_wg, w, 4, cap), "device": device} for n_wg, w, cap in shapes]
    for (n_wg, w, cap), (status, launches) in zip(shapes, fake_hip.run(calls, tmp_path)):
        assert status == 0 and "kp_pairs_main" in launches[-1][0], launches
        _, grid, block, _ = launches[-1]
        assert grid == min(n_wg, device[1] * (min(6, device[2]) if block == 256 else device[2])), (n_wg, w, cap, launches)


@pytest.mark.parametrize("cus", [128, 32])
def test_the_choice_of_a_statistics_kernel_goes_by_workgroups_per_cu(tmp_path, cus):
    """A device with fewer CUs takes as many workgroups per CU with the same kernel, on either side of every line."""
    counts = (8, 256, 264, 400, 408, 512, 520, 768, 776, 1400, 1408, 1496, 1504, 1528, 1536, 2496, 2504, 4000)
    shapes = [(2, 3, 64), (8, 5, 64), (8, 24, 128), (2, 24, 256), (2, 5, 1024), (16, 12, 128), (8, 5, 512), (8, 16, 1024), (8, 5, 2048),
              (8, 40, 128), (8, 64, 256), (7, 64, 1024), (12, 40, 512), (16, 8, 4096)]
    calls = [{"fn": "kp_trace_reduce_hdr", "trace": (n * of // 256, waves, regions, cap), "device": (of, of, 4)}
             for waves, regions, cap in shapes for n in counts for of in (256, cus)]
    done = fake_hip.run(calls, tmp_path)
    for call, (status, launches), (other_status, others) in zip(calls[::2], done[::2], done[1::2]):
        assert status == other_status == 0
        assert [x[0] for x in launches] == [x[0] for x in others], (call, launches, others)


@pytest.mark.parametrize("waves,regions,cap,last", [(2, 16, 256, 400), (2, 17, 256, 768), (7, 32, 64, 768), (12, 24, 64, 768),
                                                    (8, 24, 128, 1400), (16, 17, 64, 1400), (4, 20, 256, 768), (4, 17, 64, 256)])
def test_up_to_how_many_workgroups_four_records_go_to_a_lane(tmp_path, waves, regions, cap, last):
    """Each decoder workgroup holds one recorded workgroup then, whatever the grid."""
    calls = [{"fn": "kp_trace_reduce_hdr", "trace": (n, waves, regions, cap), "device": (0, 256, 3)} for n in (1, last, last + 1)]
    names = [kernels(launches, "kp_reduce_main")[0][0] for _, launches in fake_hip.run(calls, tmp_path)]
    assert names[0] == names[1] != names[2] and "ELi4ELi1E" in names[1], names
