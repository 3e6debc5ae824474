"""Launch grid of the z-march, on the CPU."""
from host_side import run_host


def test_every_block_of_items_has_a_workgroup(tmp_path):
    """A limit on the workgroups gives the first ones, which lie on the same XCDs,
    a second block, and the launch waits for those XCDs."""
    run_host(tmp_path, """
        for shape, kw in [((64, 3600, 33), dict(tile=12)), ((64, 3600, 33), dict(tile=4)),
                          ((128, 376, 81), {}), ((48, 40, 36), {}), ((32, 1500, 40), {})]:
            c = Ctx([fluid(*shape)], **kw)
            items = c.info().work_items
            c.step(1)
            assert get("grid") == -(-items // 32) * 8, (shape, items, get("grid"))
            c.close()
    """)
