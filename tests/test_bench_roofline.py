"""bench.py's roofline: bandwidth only from counted bytes (CPU)."""
import bench


def test_counted_traffic_is_the_bandwidth():
    r = bench.roofline_record({"hbm_bytes_per_launch": 3.2e12}, 2.4e12, 600.0)
    assert r["achieved"] == 5333.33 and r["frac"] == 0.6667 and r["traffic"] == 3.2e12
    assert r["list_element_account_gbps"] == 4000.0 and "past L2" in r["basis"]


def test_without_counters_the_account_says_what_it_is():
    r = bench.roofline_record(None, 2.4e12, 600.0)
    assert r["achieved"] == 4000.0 and r["frac"] == 0.5 and r["traffic"] is None
    assert "not traffic" in r["basis"]
