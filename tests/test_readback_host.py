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
