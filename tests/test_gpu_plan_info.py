"""famlies_plan_get_info names the route that a plan's launches take."""
import pytest

pytestmark = pytest.mark.gpu

# (m, n, k), dtype, compute -> route bits
CASES = [((256, 256, 256), "f64", "native", 64), ((950, 1000, 6000), "f64", "native", 128),
         ((1024, 16384, 512), "f64", "native", 0), ((4200, 4170, 4184), "f32", "bf16x6", 256),
         ((3500, 3480, 5580), "f32", "bf16x3", 128), ((300, 300, 300), "f64", "int8x6", 0)]


@pytest.mark.parametrize("size,dtype,compute,route", CASES)
def test_route(size, dtype, compute, route):
    import paper_2604_07311_amd as fm
    m, n, k = size
    plan = fm.famlies_plan_contract(fm.handle(0), fm.FAMLIES_F64 if dtype == "f64" else fm.FAMLIES_F32,
                                    fm._compute_code(compute), fm.make_desc((k, m), (1, k), "km"),
                                    fm.make_desc((k, n), (1, k), "kn"), fm.make_desc((n, m), (1, n), "nm"))
    info = fm.famlies_plan_get_info(plan)
    fm.famlies_plan_destroy(plan)
    assert info["kernel"] & ~63 == route, info
    assert info["kernel"] & 15 == {"native": 1, "bf16x3": 3, "bf16x6": 4, "int8x6": 14}[compute]
