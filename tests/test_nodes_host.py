"""Kernel 0's choice between a wave per row window and a thread per node, on the
CPU."""
from host_side import run_host


def test_rows_of_a_few_nodes_do_not_take_a_wave_each(tmp_path):
    """Bulk lattices with a short x axis run one node per thread (the row kernel
    would leave most of each wave idle: up to ten times the time), others one
    row window per wave; a batch goes by its sum."""
    run_host(tmp_path, """
        def grid(precision, lattice, *shapes):
            c = Ctx([fluid(*s) for s in shapes], lattice=lattice, precision=precision, kernel=0)
            c.step(1)
            assert c.info().kernel == 0 and c.info().launches_per_step == 1
            c.close()
            return get("grid")
        def per_node(*shapes):
            return sum(-(-nx * ny * nz // 256) for nx, ny, nz in shapes)
        for p in ("f64", "f32", "f16", "bf16"):
            for q in (15, 19, 27):
                for s in [(1, 300, 200), (2, 200, 100), (4, 150, 150), (8, 200, 200)]:
                    assert grid(p, q, s) == per_node(s), (p, q, s)
                for s in [(1, 20, 30), (8, 20, 20), (24, 200, 200), (64, 60, 60), (150, 40, 30)]:
                    assert grid(p, q, s) != per_node(s), (p, q, s)
        many = [(1, 300, 200), (70, 9, 8)]
        assert grid("f64", 19, *many) == per_node(*many)
        many = [(1, 30, 20), (150, 110, 90)]
        assert grid("f64", 19, *many) != per_node(*many)
    """)
