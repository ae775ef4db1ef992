"""Saved tuning caches name variants: the names that a build has written stay known."""
import pytest

from paper_2507_17301_amd import binding as nm


@pytest.mark.parametrize("shape", ["NB4_WP1_NJ1", "NB8_WP1_NJ1", "NB2_WP1_NJ1", "NB2_WP2_NJ2", "NB4_WP2_NJ2", "NB2_WP4_NJ4",
                                   "NB4_WP4_NJ4", "NB1_WP4_NJ4", "NB3_WP4_NJ4", "NB7_WP1_NJ1"])
def test_kernel_row_run_forms(shape):
    names = {nm.nm_variant_name(v) for v in range(nm.nm_variant_count())}
    assert {f"RUN_{shape}_KS{ks}" for ks in (1, 2, 3, 4)} <= names
