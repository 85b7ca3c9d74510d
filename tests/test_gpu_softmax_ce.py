"""Softmax cross-entropy (kernels_elementwise.hip) where the classes a lane holds in registers end, and on labels that are
no class."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _loss(dtype, rows, classes, logits, labels):
    import torch
    from paper_2509_23241_amd.runner import GpuStage
    st = GpuStage([(8, classes, "none")], [np.zeros((classes, 8), np.float32), np.zeros(classes, np.float32)], dtype=dtype,
                  mb=rows, n=1, stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1,
                  max_in_flight=1)
    st.forward(0, 0, torch.zeros(rows, 8, dtype=st.tdtype, device="cuda"))
    loss, dlogits = st.loss(0, logits.to(st.tdtype).cuda(), torch.from_numpy(labels.astype(np.int32)).cuda())
    out = float(loss), dlogits.double().cpu()
    st.close()
    return out


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,classes", [(1, 1), (5, 63), (7, 64), (6, 65), (9, 1023), (9, 1024), (9, 1025), (33, 1500), (4, 4097)])
def test_softmax_cross_entropy(dtype, rows, classes):
    import torch
    rng = np.random.default_rng(rows + classes)
    logits = torch.from_numpy(3 * rng.standard_normal((rows, classes))).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    labels = rng.integers(0, classes, rows)
    labels[-1] = classes - 1
    loss, dlogits = _loss(dtype, rows, classes, logits, labels)
    z = logits.double()
    logp = z - z.logsumexp(1, keepdim=True)
    want = logp.exp()
    want[torch.arange(rows), torch.from_numpy(labels)] -= 1
    want /= rows
    # exp of an fp32 difference of logits of up to 16 (rounded by 2^-21 each in the maximum, the logarithm and their sum) and
    # a sum of classes / 64 + 6 terms; bf16 results are rounded once more
    tol = 2.0 ** -21 * 3 + 2.0 ** -24 * (classes / 64 + 6)
    assert abs(loss + float(logp[torch.arange(rows), torch.from_numpy(labels)].mean())) <= tol * 16
    got = float((dlogits - want).norm())
    assert got <= (tol + (2.0 ** -9 if dtype == "bf16" else 0)) * float(want.norm()) + 1e-12


@pytest.mark.parametrize("label", [-1, 10, 1500, 2 ** 30, -2 ** 31])
@pytest.mark.parametrize("classes", [10, 1500])
def test_a_label_that_is_no_class_makes_the_loss_nan(classes, label):
    if 0 <= label < classes:
        pytest.skip("a class")
    import torch
    rng = np.random.default_rng(3)
    logits = torch.from_numpy(rng.standard_normal((6, classes))).float()
    labels = rng.integers(0, classes, 6)
    labels[2] = label
    loss, dlogits = _loss("f32", 6, classes, logits, labels)
    assert np.isnan(loss)
    want = logits.double().softmax(1)[2] / 6             # every class is another one
    assert float((dlogits[2] - want).norm()) <= 1e-5 * float(want.norm())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,classes", [(1, 16), (63, 10), (65, 2), (256, 16), (257, 16), (200, 17)])
def test_few_rows_of_few_classes(dtype, rows, classes):
    """One workgroup for all of them, up to 256 rows and 16 classes; a label that is no class makes the loss NaN there too."""
    import torch
    test_softmax_cross_entropy(dtype, rows, classes)
    for bad in (-1, classes):
        labels = np.zeros(rows, np.int64)
        labels[rows // 2] = bad
        assert np.isnan(_loss(dtype, rows, classes, torch.zeros(rows, classes), labels)[0])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,classes", [(509, 17), (512, 200), (513, 17), (516, 200), (2051, 40), (700, 1500),
                                          (513, 64), (513, 65), (512, 256), (512, 257), (5000, 3)])
def test_mean_by_the_last_workgroup_and_by_a_launch_of_its_own(dtype, rows, classes):
    """Four rows per workgroup: up to 128 workgroups (512 rows) the last to arrive forms the mean, above that a second launch; a label
    that is no class makes it NaN in both."""
    import torch
    rng = np.random.default_rng(rows + classes)
    logits = torch.from_numpy(3 * rng.standard_normal((rows, classes))).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    labels = torch.from_numpy(rng.integers(0, classes, rows))
    loss, dlogits = _loss(dtype, rows, classes, logits, labels.numpy())
    logp = logits.double().log_softmax(1)
    p, one = logp.exp(), torch.nn.functional.one_hot(labels, classes)
    tol = 2.0 ** -21 * 3 + 2.0 ** -24 * (classes / 64 + 6)          # of the logarithm of a probability, as above
    assert abs(loss + float((logp * one).sum(1).mean())) <= tol * 16
    # the difference to the label's 1 and the division by the rows round once each, a bf16 result by half a unit in the last of 8 bits
    off = p * tol * 16 + 2.0 ** -23 * (p - one).abs() + (2.0 ** -8 * (p - one).abs() if dtype == "bf16" else 0)
    assert bool(((dlogits * rows - (p - one)).abs() <= off).all())
    for row in (0, rows - 1):
        labels = np.zeros(rows, np.int64)
        labels[row] = classes
        assert np.isnan(_loss(dtype, rows, classes, torch.zeros(rows, classes), labels)[0])


@pytest.mark.parametrize("rows", [400, 600])
def test_mean_again_on_the_same_stage(rows):
    """The counter is back at zero after every call, also behind other work of the stage."""
    import torch
    from paper_2509_23241_amd.runner import GpuStage
    rng = np.random.default_rng(rows)
    st = GpuStage([(8, 100, "none")], [np.zeros((100, 8), np.float32), np.zeros(100, np.float32)], dtype="f32", mb=rows, n=1,
                  stage_index=1, num_stages=2, policy="latest", lam=0.1, lr=0.0, momentum=0.0, ring_capacity=1, max_in_flight=1)
    for j in range(4):
        logits = torch.from_numpy(3 * rng.standard_normal((rows, 100))).float().cuda()
        labels = torch.from_numpy(rng.integers(0, 100, rows).astype(np.int32)).cuda()
        st.forward(j, 0, torch.zeros(rows, 8, device="cuda"))
        loss, dlogits = st.loss(j, logits, labels)
        st.backward(j, dlogits)
        st.blend_update(j)
        want = torch.nn.functional.cross_entropy(logits.double(), labels.long())
        # as above: rounded logits of up to 16, and a sum of classes / 64 + 6 terms
        assert abs(float(loss) - float(want)) <= 16 * (2.0 ** -21 * 3 + 2.0 ** -24 * (100 / 64 + 6))
    st.close()
