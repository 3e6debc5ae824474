"""D2Q9 launches of several steps: how they are counted, on the CPU."""
from host_side import run_host


def test_even_steps_take_an_even_number_of_launches(tmp_path):
    """Each launch moves the state to the other buffer: k steps must leave it
    where k launches of one step would, at every k below a graph's."""
    run_host(tmp_path, """
        for nx, ny in [(8, 8), (160, 160), (1600, 200)]:
            c = Ctx([fluid(nx, ny, 1)], lattice=9, precision="f64", g=(0, 0, 0))
            for k in range(1, 100):
                before = get("launches")
                c.step(k)
                n = get("launches") - before
                assert 1 <= n <= k and n % 2 == k % 2, (nx, ny, k, n)
            c.close()
    """)


def test_polling_keeps_the_graph(tmp_path):
    """Repeated calls of an even number of steps, whole graphs and a remainder,
    use the graph built at the first."""
    run_host(tmp_path, """
        for k in (100, 102, 110, 130, 150, 190, 260):
            c = Ctx([fluid(160, 160, 1)], lattice=9, precision="f64", g=(0, 0, 0))
            before = get("graph_builds")
            for _ in range(6):
                c.step(k)
            assert get("graph_builds") - before == 1, k
            assert c.info().steps_done == 6 * k
            c.close()
    """)
