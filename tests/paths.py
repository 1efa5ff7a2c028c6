"""The kernels a forward runs on: the one that its sizes select, and the slab kernels
(an environment switch keeps those) where a small batch would run by columns."""


def each_path(monkeypatch, model, n):
    """Yields the name of the path that forwards of n samples take, while they
    take it; every one that there is, the slabs last."""
    monkeypatch.delenv("BITLOGIC_JUMP_LAYER", raising=False)
    path = model.path(n)
    yield path
    if path != "slab":
        monkeypatch.setenv("BITLOGIC_JUMP_LAYER", "0")
        assert model.path(n) == "slab"
        yield "slab"
        monkeypatch.delenv("BITLOGIC_JUMP_LAYER")
