"""The bounds tables that the streaming apply keeps per stream: host code only,
the HIP calls recorded in place of made (no GPU)."""
import hip_stub


def test_a_table_that_a_graph_may_hold_is_never_freed(tmp_path):
    # a captured call holds its stream's table for every replay: later calls on
    # the stream that need more (more clients, a larger shard) leave it alone,
    # and tables grow by at least half their size, so that those left behind are few
    hip_stub.run("""
assert apply(37_000_000, 8, 370_000) == 2      # the first call on the stream makes the table
first, size = get("g_last_alloc", u64), get("g_last_size", u64)
assert size >= 8 * (37_000_000 // 4096 + 2) * 4
put("g_captured_stream", 16)
assert apply(37_000_000, 8, 370_000) == 2      # captured: the graph holds that table
put("g_captured_stream", 0)
assert get("g_allocs") == 1
for n, clients in ((37_000_000, 12), (37_000_000, 64), (300_000_000, 8), (2_000_000_000, 64)):
    assert apply(n, clients, n // 8) == 2
    assert get("g_frees") == 0, (n, clients, hex(get("g_last_free", u64)))
before = get("g_allocs")
for n in range(2_000_000, 4_000_000_000, 50_000_000):
    assert apply(n, 64, n // 8, 32) == 2
assert get("g_frees") == 0 and get("g_allocs") - before < 24
""", tmp_path)


def test_a_table_may_be_made_while_another_stream_is_captured(tmp_path):
    # in the default capture mode, an allocation by a thread in the same mode is
    # refused and breaks the capture, whatever stream it is for
    hip_stub.run("""
put("g_other_capture", 1)
for clients in (4, 12, 64):
    assert apply(37_000_000, clients, 1_000_000) == 2
    assert get("g_refused") == 0, clients
    assert get("g_mode") == 0              # and the thread's own mode is as before
""", tmp_path)
