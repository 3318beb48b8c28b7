"""The workspace a context needs (inpaint_workspace_bytes; host only): a server
admits jobs by it, so it does not grow."""
import pytest

B = pytest.importorskip("paper_1403_4238_amd.binding")


# Radius 4, no log: the bytes that the SIMT search's contexts have needed since
# they have had one, with the original and with the current source region.
@pytest.mark.parametrize("width,height,original,current", [
    (17, 17, 111872, 112384),
    (64, 48, 247808, 250880),
    (400, 300, 4862720, 4982784),
    (640, 480, 12022016, 12329216),
    (1920, 1080, 78662656, 80736256),
    (30000, 17, 31166720, 31676928),
    (6000, 4000, 898968576, 922968576),
])
@pytest.mark.parametrize("path", [B.PATH_AUTO, B.PATH_SIMT, B.PATH_MFMA])
def test_workspace_does_not_grow(width, height, original, current, path):
    assert B.inpaint_workspace_bytes(width, height, B.make_params(4, path=path)) <= original
    if path != B.PATH_MFMA:
        p = B.make_params(4, path=path, source_policy=B.SOURCE_CURRENT)
        assert B.inpaint_workspace_bytes(width, height, p) <= current
