"""Route workspace sizes (host only)."""
import paper_2608_18410_amd as rs


def test_workspace_size_grows_with_the_batch():
    """A workspace sized for a batch holds every smaller one (both routers)."""
    for router in (rs.Router(rs.MLP2, 8, {}, d_e=128, Hr=128), rs.Router(rs.ADDITIVE, 6, {})):
        for T in (1, 81, 177, 2048):
            sizes = [rs.route_workspace_size(B, T, 16, 4096, router) for B in range(1, 140)]
            assert sizes == sorted(sizes)
