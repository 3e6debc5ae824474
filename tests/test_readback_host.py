"""Host side of the readback (state and permeability), on the CPU."""
from host_side import run_host


def test_block_and_events_are_visible_to_the_host(tmp_path):
    """The pinned block asks for coherence, a slot's event for a release to the
    system (values of hipHostMallocPortable, hipHostMallocCoherent,
    hipEventDisableTiming and hipEventReleaseToSystem in the HIP API)."""
    run_host(tmp_path, """
        c = Ctx([fluid(8, 4, 4)])
        st, d, u = c.read()
        assert st == 0
        assert get("pinned_flags") & 0xffffffff == 0x1 | 0x40000000
        assert get("event_flags") & 0xffffffff == 0x2 | 0x80000000
        c.close()
    """)


def test_no_pinned_memory(tmp_path):
    """Without pinned memory the fields and the permeability come through the
    workspace (here the staging area's own values: kernels do nothing)."""
    run_host(tmp_path, """
        for shape in [(8, 4, 4), (160, 128, 150)]:      # one chunk, two
            c = Ctx([fluid(*shape)], precision="f64")
            put("refuse_pinned", 1)
            before = get("launches")
            c.mem[:] = 7.0      # also the staging area (and the flag of non-finite values,
            st, d, u = c.read() # which is cleared first)
            assert st == 0
            assert np.all(d == 7.0) and np.all(u == 7.0)
            chunks = -(-d.size // (1 << 21))
            assert get("launches") - before == chunks
            assert lib.tau1_moments_drho(c.p, 0, None, u.ctypes.data) == 0
            assert c.permeability() in (0, tau1.TAU1_E_NONFINITE)
            put("refuse_pinned", 0)
            assert c.read()[0] == 0
            c.close()
        assert get("pinned") > 0
    """)


def test_pinned_blocks_go_back_without_a_wait_of_the_caller(tmp_path):
    """hipHostFree waits for every stream of the device: neither the last
    context's end nor a read that finds the pool full calls it on the caller's
    thread, and every block is given back."""
    run_host(tmp_path, """
        import threading, time
        for rounds in range(3):
            cs = [Ctx([fluid(16, 16, 40 + 8 * i)]) for i in range(4)]
            ts = [threading.Thread(target=lambda c=c: [c.read() for _ in range(20)]) for c in cs]
            for t in ts: t.start()
            for t in ts: t.join()
            for c in cs: c.close()
            deadline = time.time() + 20
            while get("freed") != get("pinned") and time.time() < deadline:
                time.sleep(0.01)
            assert get("pinned") > 0 and get("freed") == get("pinned")
        assert get("freed_here") == 0
    """)


def test_reads_under_capture_launch_nothing(tmp_path):
    """A read fails under capture (its wait is refused there); its kernels, which
    write to a pinned block of the pool, must not end up in the captured graph."""
    run_host(tmp_path, """
        for call in ("read", "permeability"):
            c = Ctx([fluid(8, 4, 4)])
            put("capturing", 1)
            before = get("launches")
            st = getattr(c, call)()
            st = st[0] if isinstance(st, tuple) else st
            assert st == tau1.TAU1_E_HIP
            assert get("launches") == before
            put("capturing", 0)
            c.close()
    """)


def test_events_are_made_with_the_context(tmp_path):
    """The readback's events are made by tau1_create, where the context's device
    is the current one, and not by the first read."""
    run_host(tmp_path, """
        c = Ctx([fluid(8, 4, 4)])
        made = get("events")
        assert made > 0
        assert c.read()[0] == 0
        assert get("events") == made
        c.close()
    """)
