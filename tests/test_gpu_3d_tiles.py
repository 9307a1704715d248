"""The 3D faces' solve works on 8 x 8 tiles of rows with four rows of halo: faces smaller than the
halo, one tile exactly, one row more, several tiles, against the FP64 oracle (tolerances as there)."""
import pytest

from test_gpu_3d import RELAX, compare3, drifting_pulse

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc,recon,precision", [
    (["lodi_relax", "cbc_relax"], None, "fp64"), (["cbc", "zg"], None, "fp32dev"), (["zg", "lodi"], "neep", "fp64")])
@pytest.mark.parametrize("ny,nz", [(4, 4), (8, 8), (9, 5), (4, 17), (19, 16)])
def test_3d_face_tiles(ny, nz, bc, recon, precision):
    nx = 14
    compare3("tiles", nx, ny, nz, bc, drifting_pulse(nx, ny, nz, (7, ny / 3, nz / 2), width=2.0), precision, [1, 2, 5, 12],
             relax=RELAX, recon=recon)


@pytest.mark.parametrize("axis,dims,recon", [(0, (14, 193, 170), None), (1, (9, 14, 11), "neep")])
def test_3d_face_tiles_limits(axis, dims, recon):
    """Faces on the other side of the tile count's limit (stage by stage), and a rotated axis."""
    nx, ny, nz = dims
    compare3("tiles-limit", nx, ny, nz, ["lodi_relax", "cbc"], drifting_pulse(nx, ny, nz, (nx / 2, ny / 3, nz / 2), width=2.0),
             "fp64", [1, 3], relax=RELAX, recon=recon, axis=axis)
