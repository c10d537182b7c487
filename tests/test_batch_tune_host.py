"""The batch autotuner's default candidates, without a GPU: the automatic
workgroup size is among them, so that tuning never ends slower than not
tuning."""


class Recorder:
    """Stands in for a Batch: times each configuration by a table."""

    def __init__(self, ms):
        self.ms, self.configs = ms, []

    def _full_grid(self):
        return 1024

    def config(self, threads=0, grid=0, use_graph=True):
        self.configs.append((threads, grid, use_graph))

    def run(self, n_mcs, p, q):
        pass

    def sync(self):
        pass

    def timing(self, enable=True):
        pass

    def get_timing(self):
        return {"ms": self.ms(*self.configs[-1])}


def test_automatic_size_is_a_candidate():
    import paper_1705_01022_amd as okpz

    r = Recorder(lambda threads, grid, graph: 1.0 if (threads, grid) == (0, 0) else 2.0)
    got = okpz.Batch.tune(r, [1], [1.0], [0.0])
    assert got["best"] == (0, 1.0, True)
    assert r.configs[-1] == (0, 0, True)


def test_a_faster_fixed_size_is_kept():
    import paper_1705_01022_amd as okpz

    r = Recorder(lambda threads, grid, graph: 1.0 if threads == 128 else 2.0)
    got = okpz.Batch.tune(r, [1], [1.0], [0.0])
    assert got["best"] == (128, 1.0, True) and r.configs[-1] == (128, 0, True)
    assert set(got["times_ms"]) >= {(0, 1.0, True), (256, 1.0, True), (512, 1.0, True), (256, 0.5, True),
                                    (256, 1.0, False)}
