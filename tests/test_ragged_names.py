"""Ragged shape names of earlier tune files keep working."""
import paper_2603_27569_amd as sf


def test_retired_ragged_shape_name_is_accepted():
    try:
        sf.fft_tune_set_ragged(16384, "ragged_n16384_e32c2_r8")
        assert sf.fft_tune_query_ragged(16384) == "ragged_n16384_e32c2_r32"
    finally:
        sf.fft_tune_clear_ragged()
