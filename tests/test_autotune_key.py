"""A tuned launch shape is looked up by everything that decides what the candidates
mean: batches of one shape but other flags, and other libraries, have keys of
their own."""
from paper_1311_4527_amd import autotune, instances as I
from paper_1311_4527_amd import twa as T


def test_key_tells_flags_and_libraries_apart(tmp_path, monkeypatch):
    insts = [I.circle_swap(6, 0.05, 2, seed=k) for k in range(3)]
    for k in range(2):
        (tmp_path / f"lib{k}.so").write_bytes(b"library %d" % k)
    keys = set()
    for k in range(2):
        monkeypatch.setattr(T, "LIB_PATH", str(tmp_path / f"lib{k}.so"))
        for flags in (0, T.TWA_F_DENSE, T.TWA_F_ADMM):
            keys.add(autotune.cache_key("gpu", insts, flags, 20))
    assert len(keys) == 6
    assert autotune.cache_key("gpu", insts[::-1], T.TWA_F_ADMM, 20) in keys  # (the order of instances is no matter)
    assert autotune.cache_key("gpu", insts[:2], T.TWA_F_ADMM, 20) not in keys
