"""The per-voxel passes behind the tests that use the library's default
configuration.  A default handle solves over the grey levels; here the same
tests run with every handle that would, on the per-voxel pass of the persistent
driver in its default shape instead (the grid named, which is how a caller asks
for it): the large-volume sweep with FP64 and compensated FP32 cross-block sums
(48 cases), cluster counts, fuzziness, ragged sizes, special cases, steps,
asynchronous solves, random and learned starts."""
import pytest

from phantom import PhantomParams, phantom
from tests.test_gpu_async import (test_async_equals_sync, test_async_many_sizes,  # noqa: F401
                                  test_async_mixed_with_sync_calls)
from tests.test_gpu_config3 import test_large_volume_sweep, torch_dev  # noqa: F401
from tests.test_gpu_learn import (test_invalid_network_output_selects_the_plain_start,  # noqa: F401
                                  test_solve_warm_follows_algorithm_1_and_falls_back,
                                  test_warm_start_in_kernel_and_launched)
from tests.test_gpu_parity import (check_against_literal, test_bitwise_deterministic,  # noqa: F401
                                   test_cluster_counts_m2, test_constant_image, test_fewer_voxels_than_clusters,
                                   test_fuzziness, test_given_init, test_iterate_in_steps_equals_solve,
                                   test_labels_to_misaligned_buffer, test_max_iter_not_converged,
                                   test_ragged_sizes_and_offsets, test_slice_200x200_c4_m2, test_timing_flag,
                                   test_two_levels_exact, test_volume_181x217x181, test_volume_512x512x256,
                                   test_volume_64x128x128_c4_m2, test_volume_kahan_only,
                                   test_voxel_on_centroid_gets_full_membership)
from tests.test_gpu_random import (test_paper_protocol_slice, test_paper_protocol_stepwise,  # noqa: F401
                                   test_paper_protocol_tight_eps, test_paper_protocol_tiny_and_max_iter,
                                   test_paper_protocol_volume_unaligned, test_seed_changes_start)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def per_voxel(monkeypatch):
    import paper_1601_00072_amd as pkg

    class VoxelFCM(pkg.FCM):
        def __init__(self, *a, **kw):
            super().__init__(*a, **kw)
            self.set_tuning()

        def set_tuning(self, **kw):
            super().set_tuning(**kw)
            t = self.tuning
            if t["driver"] == 2 and t["grid"] == 0:  # over the grey levels
                super().set_tuning(driver=0)
                super().set_tuning(**{**kw, "driver": 2, "grid": self.tuning["grid"]})
            assert self.tuning["grid"] > 0

    monkeypatch.setattr(pkg, "FCM", VoxelFCM)


@pytest.mark.parametrize("driver,exchange", [(0, 0), (1, 0), (2, 0), (2, 1), (2, 2)])
@pytest.mark.parametrize("grid", [0, 3, 300])
@pytest.mark.parametrize("C,m", [(4, 2.0), (7, 1.5), (3, 2.5)])
def test_compensated_sums(torch_dev, driver, exchange, grid, C, m):  # noqa: F811
    """FCM_F_KAHAN_ONLY in every per-voxel driver and exchange that takes it,
    with fewer rows than threads of the reduction and with more."""
    print("CASE compensated sums, driver", driver, "exchange", exchange, "grid", grid, "C", C, "m", m, flush=True)
    x = phantom(PhantomParams(shape=(31, 64, 63), seed=6))
    check_against_literal(torch_dev, x, C, m=m, kahan_only=True,
                          tuning=dict(driver=driver, exchange=exchange, grid=grid))
