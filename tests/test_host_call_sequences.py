"""What the library's calls ask of the runtime, seen on the CPU: libllr.so against
a recorder in the runtime's place (no kernel runs)."""
from tests.hip_recorder import run


def test_beta_c_noalloc_allocates_nothing(tmp_path):
    """Neither device nor host memory, also where inputs exceed the pinned buffer
    (n = 5000); the allocating call is there to show that the counters count."""
    got = run(tmp_path, '''
h = context()
result = []
for n in (128, 5000):
    c, a = 1000.0 + np.arange(n), np.full(n, 1.01)
    bc, pk = C.c_double(), C.c_double()
    for f in (L.llr_beta_c, L.llr_beta_c_noalloc):
        rec.rec_reset()
        st = f(h, dptr(c), dptr(a), n, 1.0, 1e4, 1.0, 1.01, 1e-5, 1e-9, C.byref(bc), C.byref(pk))
        result.append([st, rec.rec_news(), sum(k[0] in ("hipMalloc", "hipHostMalloc") for k in calls())])
''')
    assert [g[0] for g in got] == [0, 0, 0, 0]
    assert got[0][2] == 1 and got[2][2] == 1
    assert got[1][1:] == [0, 0] and got[3][1:] == [0, 0], got


def test_prob_peaks_room_follows_the_intervals(tmp_path):
    """n intervals have fewer than n interior maxima, so a caller's larger max_peaks
    asks for no more memory than n does, on either side."""
    got = run(tmp_path, '''
result = []
n = 40
c, a = 1000.0 + np.arange(n), np.full(n, 1.01)
E, lp, nf = np.zeros(n), np.zeros(n), C.c_int()
for peaks in (n, 1 << 22):
    h = context()
    rec.rec_reset()
    st = L.llr_prob_peaks(h, dptr(c), dptr(a), n, 1.0, 1.01, peaks, dptr(E), dptr(lp), C.byref(nf))
    result.append([st, rec.rec_new_max(), sum(k[3] for k in calls() if k[0] != "launch")])
''')
    assert got[0] == got[1], got


def test_error_in_halves_leaves_no_work_on_the_second_stream(tmp_path):
    """Each event call of an iteration in two halves made to fail in turn: the call
    reports it, and waits for what it has put on its second stream."""
    got = run(tmp_path, '''
result = []
for order in (llr.SWEEP_GROUPED, llr.SWEEP_INTERLEAVED, llr.SWEEP_STAGGERED):
    h = context(llr.FP32, [(16, 25)], order, n_th=2, n_a=4)
    assert L.llr_rm_begin(h) == 0
    rec.rec_reset()
    assert L.llr_rm_step(h, 1) == 0
    done = calls()
    for op in ("hipEventRecord", "hipStreamWaitEvent"):
        for at in range(sum(k[0] == op for k in done)):
            rec.rec_reset()
            rec.rec_fail(op.encode(), at)
            st = L.llr_rm_step(h, 1)
            left = 0
            for kind, name, stream, _ in calls():
                if stream != 0x77 and kind == "launch": left += 1
                if stream != 0x77 and kind == "hipStreamSynchronize": left = 0
            result.append([st, left])
''')
    assert len(got) > 60 and all(st == -3 for st, _ in got), got
    assert all(left == 0 for _, left in got), got


def test_training_workspace_does_not_grow_with_epochs(tmp_path):
    """Beyond the losses themselves, 8 bytes an epoch."""
    got = run(tmp_path, '''
result = []
fp = C.POINTER(C.c_float)
n = 4096
w, u, il, a = np.zeros(llr.N_PARAMS, np.float32), np.full(n, 0.6, np.float32), np.full(n, 0.1, np.float32), np.ones(n)
for epochs in (1000, 5000):
    h = context()
    rec.rec_reset()
    hist = np.zeros(epochs)
    st = L.llr_mlp_train(h, w.ctypes.data_as(fp), u.ctypes.data_as(fp), il.ctypes.data_as(fp), dptr(a), n, epochs, 1e-3,
                         1, dptr(hist))
    result.append([st, sum(k[3] for k in calls() if k[0] == "hipMalloc")])
''')
    assert got[0][0] == got[1][0] == 0
    assert got[1][1] - got[0][1] == 8 * 4000, got


def test_short_runs_stay_whole(tmp_path):
    """A run of a few sweeps is not split into halves: the second half has to wait for
    the first to get ahead, and no later sweep makes up for it."""
    got = run(tmp_path, '''
result = {}
for name, prec, lats, order, counts in (("g", llr.FP64, [(12, 20)], llr.SWEEP_GROUPED, (1, 2, 5, 6)),
                                        ("i", llr.FP64, [(12, 20)], llr.SWEEP_INTERLEAVED, (1, 3, 4)),
                                        ("G", llr.FP32, [(18, 96)], llr.SWEEP_GROUPED, (1, 2)),
                                        ("I", llr.FP32, [(18, 96)], llr.SWEEP_INTERLEAVED, (1,))):
    streams = []
    for n in counts:
        h = context(prec, lats, order, n_th=0, n_a=n)
        assert L.llr_rm_begin(h) == 0
        for f in (lambda: L.llr_sweeps(h, n, 3, llr.MODE_FREE, None), lambda: L.llr_rm_step(h, 1)):
            rec.rec_reset()
            assert f() == 0
            # launches of a captured sweep go to the capturing stream
            capturing = [k[2] for k in calls() if k[0] == "hipStreamBeginCapture"]
            streams.append(len({k[2] for k in calls() if k[0] == "launch" and k[2] not in capturing}))
        L.llr_destroy(h)
    result[name] = streams
''')
    assert got == {"g": [1, 1, 1, 1, 1, 1, 2, 2], "i": [1, 1, 1, 1, 2, 2], "G": [1, 1, 2, 2], "I": [2, 2]}, got


def test_staggered_order_of_single_chains_needs_one_stream(tmp_path):
    """Without a second half there is nothing to fork: iterations replay their captured
    sweeps, and direct launches stay on the context's stream."""
    got = run(tmp_path, '''
h = context(llr.FP32, [(10, 1), (12, 1)], llr.SWEEP_STAGGERED, n_th=1, n_a=3)
assert L.llr_rm_begin(h) == 0
rec.rec_reset()
assert L.llr_rm_step(h, 1) == 0 and L.llr_sweeps(h, 2, 3, llr.MODE_FREE, None) == 0
k = calls()
result = [sum(x[0] == "hipGraphLaunch" for x in k), sum(x[0] == "hipStreamWaitEvent" for x in k)]
''')
    assert got == [4, 0], got


def test_interleaved_sweeps_of_l8_leave_lds_where_class_passes_are_faster(tmp_path):
    got = run(tmp_path, '''
result = {}
def resident(h):
    rec.rec_reset()
    assert L.llr_rm_begin(h) == 0 and L.llr_rm_step(h, 1) == 0
    names = [k[1] for k in calls() if k[0] == "launch"]
    chain = any("k_chain" in n for n in names)
    assert chain != any("k_hb" in n for n in names)
    return chain
for ex, counts in ((1, (1, 127, 128, 256, 257)), (0, (1, 512, 513))):
    for n in counts:
        result["%d %d" % (ex, n)] = resident(context(llr.FP32, [(8, n)], llr.SWEEP_INTERLEAVED, replica_exchange=ex))
# other orders, smaller lattices and the rest of the calls are kept in LDS
h = context(llr.FP32, [(8, 3)], llr.SWEEP_GROUPED, replica_exchange=1)
result["grouped"] = resident(h)
result["L=6"] = resident(context(llr.FP32, [(6, 3)], llr.SWEEP_INTERLEAVED, replica_exchange=1))
''')
    assert got == {"1 1": False, "1 127": False, "1 128": True, "1 256": True, "1 257": False,
                   "0 1": True, "0 512": True, "0 513": False, "grouped": True, "L=6": True}, got
