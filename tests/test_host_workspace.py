"""What a state's workspace holds (host only)."""
import pytest

from conftest import cube

B = pytest.importorskip("paper_2203_00925_amd.binding")


def test_matrix_free_workspace_holds_nothing_of_the_matrix():
    """Per stored entry its column, value, FP32 value and local column (18
    bytes); per halo entry of the stored product's tiles its entity."""
    m = cube(12, 3)
    full, free = (B.Mesh.from_cube(m, no_matrix=k).info for k in (False, True))
    assert free.halo_entries == full.halo_entries and free.matrix_padded == 0
    assert full.ws_bytes - free.ws_bytes >= 18 * full.matrix_padded + 4 * full.halo_entries
