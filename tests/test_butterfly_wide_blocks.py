"""The plan of the GPU test of wide blocks has what it names: child blocks of more
than 64 dense rows, and of up to 64.  Host-only."""
from test_plan_file_tables import File


def test_block_widths(tmp_path):
    from paper_1110_4874_amd import sht
    path = str(tmp_path / "p.plan")
    sht.Plan(511, 200, 1e-11, max_levels=3, host_only=True).save(path)
    dense = File(path).array("node_i", "i4").reshape(-1, 16)[:, 4:6]
    assert (dense > 64).sum() > 1000 and (dense <= 64).sum() > 1000
