"""The autotune cache tells a fixed tile from the automatic choice, which goes by
a tile's name but has segments of its own length, on the CPU."""
from host_side import run_host


def test_cached_choice_is_the_one_applied(tmp_path):
    run_host(tmp_path, """
        cache = sys.argv[3]
        seen = 0
        for shape in [(64, 48, 40), (128, 60, 50), (96, 90, 72), (256, 100, 96), (160, 64, 150)]:
            def items(**kw):
                c = Ctx([fluid(*shape)], **kw)
                c.mem[:] = 0.0
                inf = c.info()
                c.close()
                return inf.tile, inf.work_items
            tile, auto = items()
            own = items(tile=tile)[1]
            if own == auto:
                continue
            seen += 1
            bucket = 1
            while bucket < np.prod(shape):
                bucket *= 2
            line = f"tau1 gfx950 q19 p1 n{bucket} tile %s ms 0.5"
            print(line % tile, file=open(cache, "w"))
            assert items(tune_cache=cache) == (tile, own)      # a fixed tile is applied
            print(line % "auto", file=open(cache, "w"))
            assert items(tune_cache=cache) == (tile, auto)     # ... the automatic choice too
            # the tuner's record of an automatic winner (all trials take the same
            # time here, and the automatic choice is tried first)
            open(cache, "w").close()
            c = Ctx([fluid(*shape)], tune_cache=cache)
            assert lib.tau1_autotune(c.p, 2) == 0
            assert c.info().work_items == auto
            c.close()
            assert "tile auto" in open(cache).read()
            assert items(tune_cache=cache) == (tile, auto)
        assert seen >= 2
    """, tmp_path / "tune")
