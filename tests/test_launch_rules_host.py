"""What the host side launches, recorded without a GPU: grids against the limits
of their kernels, and which kernels a call takes."""
import recorder


def test_histogram_bins_of_a_workgroup_cannot_overflow():
    # each of a workgroup's references adds up to n - 1 pairs to one 32-bit bin
    got = recorder.run("""
result = []
for n in (1, 2, 1000, 1024, 1025, 48077, 2097152, 2097153, 3000000, 6000000):
    pos = np.zeros((n, 3))
    pos[:, 0] = np.arange(n)
    with scmd.Simulation([0, n], pos) as sim:
        records()
        sim.rdf(0, 1.0, 16)
        result.append([n] + [r[2] for r in records() if r[0] == "launch" and "k_rdf_hist" in r[1]])
""")
    for n, groups in got:
        per_group = -(-n // groups)
        assert per_group * (n - 1) < 2**32, (n, groups)


def test_an_evaluation_takes_the_kernels_of_the_run():
    # so that compute() between two calls of step() changes no bit of what follows
    got = recorder.run("""
result = []
for sizes in ([13], [96], [97], [147], [152], [153], [2243], [3501], [150] * 16, [96] * 16):
    off = np.concatenate([[0], np.cumsum(sizes)])
    with scmd.Simulation(off, np.concatenate([cluster(n) for n in sizes])) as sim:
        sim.compute()
        evaluation = sorted({r[1] for r in records()})
        sim.step(1)
        result.append([sizes, evaluation, sorted({r[1] for r in records()})])
""")
    family = lambda names: {f for n in names for f in ("k_resident", "k_row_", "k_sym_") if f in n}
    for sizes, evaluation, run in got:
        assert family(evaluation) == family(run) and len(family(run)) == 1, sizes


def test_batches_above_152_atoms_stay_resident_only_when_they_fill_the_chip():
    # one workgroup per cluster takes as long for 16 clusters as for 256; the row
    # sweeps of a few are faster (16 x 190 atoms 10.3 us per step against 13.5)
    got = recorder.run("""
result = []
for sizes in ([152] * 2, [152] * 16, [153] * 16, [190] * 16, [190] + [13] * 15, [190] * 42, [190] * 48, [191] * 48,
              [190] + [55] * 511):
    off = np.concatenate([[0], np.cumsum(sizes)])
    with scmd.Simulation(off, np.concatenate([cluster(n) for n in sizes])) as sim:
        records()
        sim.step(1)
        result.append([any("k_resident" in r[1] for r in records())])
""")
    assert [r[0] for r in got] == [True, True, False, False, False, False, True, False, True]


def test_row_sweeps_on_request_have_eight_wavefronts_unless_told_otherwise():
    got = recorder.run("""
result = []
for n in (700, 2560, 2561, 4096):
    for tuning in (dict(pairs=3), dict(pairs=3, waves_j=8), dict(pairs=3, waves_j=16)):
        with scmd.Simulation([0, n], cluster(n), tuning=tuning) as sim:
            records()
            sim.step(1)
            result.append([n, tuning.get("waves_j", 0), sorted({r[3] // 64 for r in records() if r[0] == "launch" and "k_row" in r[1]})])
""")
    assert all(waves == [asked or 8] for _, asked, waves in got), got


def test_the_lds_limit_of_a_kernel_does_not_depend_on_the_call():
    # the limit belongs to the kernel: a smaller one, set by a context on another
    # thread, must not come between a context's own setting and its launch
    got = recorder.run("""
result = []
for n in (13, 48, 49, 96, 97, 152, 700, 2243, 2500, 2600, 3000):
    for kw in ({}, dict(precision="mixed"), dict(params=dict(n=12, m=6)), dict(rc=8.8)):
        with scmd.Simulation([0, n], cluster(n), **kw) as sim:
            sim.step(2)
            for bins in (100, 20000, 32768):
                sim.rdf(0, 0.01, bins)
        result += records()
""")
    limits, lds = {}, {}
    for kind, kernel, *nums in got:
        if kind == "limit":
            limits.setdefault(kernel, set()).add(nums[0])
        else:
            lds[kernel] = max(lds.get(kernel, 0), nums[2])
    for family in ("k_resident", "k_row_density", "k_row_force", "k_rdf_hist", "k_cell_sweep"):
        assert any(family in k for k in limits), family
    for kernel, bytes_ in lds.items():
        assert len(limits.get(kernel, {65536})) == 1, kernel
        assert bytes_ <= min(limits.get(kernel, {65536})), kernel


def test_cell_list_memory_of_a_sparse_box():
    # two atoms 1000 A apart span about 1.6 million cells; a cell needs its
    # cluster, count, start, cursor and place (4 bytes each) and a slot of 32
    # bytes for its sums, records are for cells that can hold atoms
    got = recorder.run("""
pos = np.array([[0.0, 0.0, 0.0], [1000.0, 1000.0, 1000.0]])
with scmd.Simulation([0, 2], pos, rc=8.8) as sim:
    before = rec.rec_device_bytes()
    sim.compute()
    cells = max(r[2] for r in records() if "k_cell_order" in r[1])
    result = [cells, rec.rec_device_bytes() - before]
""")
    cells, added = got
    assert cells > 10**6
    assert added <= 52 * cells + 65536, added / cells


def test_symmetric_items_of_middle_sizes_fit_three_per_compute_unit():
    # one j tile per item while that is at most 768 items, then two (1024 items
    # asked for give two from 66 tiles on)
    got = recorder.run("""
result = []
for n in (3073, 3520, 3521, 3600, 4096, 4160, 4161, 4480):
    with scmd.Simulation([0, n], cluster(n), tuning=dict(pairs=2)) as sim:
        sim.compute()
        result.append([n, max(r[2] for r in records() if r[0] == "launch" and "k_sym_force" in r[1])])
""")
    assert all(items <= 768 for _, items in got), got


def test_auto_plans_do_not_fall_behind_the_library_s_own():
    # a plan timed at 2243 atoms kept single clusters of 2049 to 4096 on 8
    # wavefronts and off the symmetric sweeps; it holds near 2243 only
    got = recorder.run("""
result = []
for n in (2060, 2600, 3501, 4096, 13, 147, 9000, 40000):
    off = np.array([0, n])
    own = []
    for tuning in (None, "auto"):
        with scmd.Simulation(off, cluster(n), tuning=tuning) as sim:
            records()
            sim.step(1)
            own.append(sorted({tuple(r) for r in records() if r[0] == "launch"}))
    result.append([n, own[0] == own[1]])
""")
    assert all(same for _, same in got), got


def test_the_autotuner_times_the_library_s_own_plan():
    from paper_1210_3559_amd import autotune, inputs
    for name in ("ni147_nve", "ni2243_cooling", "batch256"):
        assert {} in autotune.tunings(inputs.by_name(name))
    rows = [dict(tuning={}, ms_per_step=1.0), dict(tuning=dict(pairs=3), ms_per_step=1.02),
            dict(tuning=dict(pairs=2), ms_per_step=1.5)]
    assert autotune.pick(rows)["tuning"] == dict(pairs=3)  # within the noise: the plan itself is recorded
    rows[0]["ms_per_step"] = 0.5
    assert autotune.pick(rows)["tuning"] == {}
    assert autotune.pick([dict(tuning=dict(cell_skin=0.4), ms_per_step=1.0)])["tuning"] == dict(cell_skin=0.4)


def test_middle_batches_take_the_sweeps_that_are_faster():
    # the batches that the row sweeps run faster (us per step against symmetric)
    # and those they do not, at alike numbers of pairs
    got = recorder.run("""
result = []
for sizes in ([800] * 8, [1000] * 6, [1000] * 8, [1300] * 4, [1700] * 3, [2000] * 2, [500] * 27, [400] * 42,
              [2243] + [55] * 20, [1500] * 3, [1400] * 4, [700] * 13, [400] * 38, [1000] * 10, [2400] * 2, [2057] * 4):
    off = np.concatenate([[0], np.cumsum(sizes)])
    with scmd.Simulation(off, np.concatenate([cluster(n) for n in sizes])) as sim:
        records()
        sim.step(1)
        result.append([sizes[0], len(sizes), any("k_row" in r[1] for r in records())])
""")
    assert [row for *_, row in got] == [True] * 9 + [False] * 7, got


def test_single_clusters_change_sweeps_where_both_take_as_long():
    got = recorder.run("""
result = []
for precision in ("fp64", "mixed"):
    for n in (3072, 3073, 3520, 3521, 4096, 4097):
        with scmd.Simulation([0, n], cluster(n), precision=precision) as sim:
            records()
            sim.step(1)
            result.append(any("k_row" in r[1] for r in records()))
""")
    assert got == [True, True, True, False, False, False, True, True, True, True, True, False]


def test_general_exponents_leave_the_resident_kernel_earlier():
    # the power chains take one CU longer: 147 atoms 14.9 us per step, row sweeps 9.5
    got = recorder.run("""
result = []
for precision in ("fp64", "mixed"):
    for n, k in ((96, 1), (97, 1), (152, 1), (152, 32), (190, 64), (190, 72), (152, 72)):
        with scmd.Simulation(np.arange(k + 1) * n, np.tile(cluster(n), (k, 1)), precision=precision,
                             params=dict(n=12, m=6, c=144.41)) as sim:
            records()
            sim.step(1)
            result.append(any("k_resident" in r[1] for r in records()))
""")
    assert got == 2 * [True, False, False, False, False, True, True]


def test_histogram_workgroups_follow_the_bins_and_the_references():
    # (atoms, bins, workgroups): one per atom, four per CU, what the LDS leaves room
    # for, eight references each
    want = [(100, 400, 100), (2057, 400, 1024), (1000, 20000, 512), (1000, 32768, 256), (48077, 400, 6010),
            (48077, 20000, 6010), (48077, 32768, 256)]
    got = recorder.run(f"""
result = []
for n, bins, _ in {want!r}:
    pos = np.zeros((n, 3))
    pos[:, 0] = np.arange(n)
    with scmd.Simulation([0, n], pos) as sim:
        records()
        sim.rdf(0, 1.0, bins)
        result.append([n, bins] + [r[2] for r in records() if r[0] == "launch" and "k_rdf_hist" in r[1]])
""")
    assert list(map(tuple, got)) == want


def test_getters_pack_once_where_the_staging_area_holds_the_result():
    # results that fit half the staging area, all of it, and neither; densities of
    # more than 16 KiB are copied without a kernel
    got = recorder.run("""
result = []
for n in (1, 2048, 2049, 5461, 5462, 10922, 10923, 40000):
    pos = np.zeros((n, 3))
    pos[:, 0] = np.arange(n)
    with scmd.Simulation([0, n], pos, rc=8.8) as sim:
        sim.compute()
        records()
        launches = []
        for get in (sim.positions, sim.density):
            get()
            launches.append(len([r for r in records() if r[0] == "launch"]))
        result.append([n] + launches)
""")
    for n, xyz, density in got:
        assert xyz == (1 if 24 * n <= 1 << 18 else -(-n // ((1 << 17) // 24))), n
        assert density == (1 if n <= 2048 else 0), n
