"""Which form of the apply a call takes: host code only, the launches recorded
in place of made (no GPU)."""
import hip_stub


def test_up_to_8_clients_stream_from_an_entry_per_64_parameters(tmp_path):
    # whatever the size of the shard: pushes this dense may lie in few rows, where
    # the scattered form is up to 20 times slower, and streaming costs the same anywhere
    hip_stub.run("""
for n in (2_000_000, 9_700_000, 1 << 24, (1 << 24) + 1, 37_000_000, 2_000_000_000):
    for clients in (1, 2, 4, 8):
        dense = -(-n // (64 * clients))
        assert apply(n, clients, dense) == 2, (n, clients)
        assert apply(n, clients, n // (64 * clients) - 1) == 1, (n, clients)
""", tmp_path)


def test_more_clients_stream_when_denser_on_large_shards(tmp_path):
    hip_stub.run("""
for clients in (9, 16, 64):
    for n, per in ((9_700_000, 128), (1 << 24, 128), ((1 << 24) + 1, 48), (37_000_000, 48)):
        dense = -(-n // (per * clients))
        assert apply(n, clients, dense) == 2, (n, clients)
        assert apply(n, clients, n // (per * clients) - 1) == 1, (n, clients)
    put("g_captured_stream", 16)
    assert apply(9_700_000, clients, 100_000) == 1   # captured calls of more than 8 never stream
    put("g_captured_stream", 0)
""", tmp_path)
