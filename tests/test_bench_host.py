"""The batch benchmark says which launches its tuned strip heights belong to."""
import bench


def test_tuning_summary_names_the_launches():
    assert bench.tuning_summary(None, 1.0, "f32") is None
    one, two = (bench.tuning_summary([2, 3, 3], 1.0, s) for s in ("f16local", "f32"))
    assert one["rows_of"] == "the step launches" and "single-step" in two["rows_of"]
    assert one["rows_histogram"] == {"2": 1, "3": 2}
