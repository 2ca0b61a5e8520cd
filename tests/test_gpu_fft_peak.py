"""The measured double-precision peak (vlp_measure_fft_peak): rates are plausible
for the instruction count of a butterfly, the CMux mix lies between its two
parts, and a bad device is an argument error."""
import pytest

pytestmark = pytest.mark.gpu


def test_measured_butterfly_rates():
    from paper_2506_12761_amd import vlp
    r = vlp.vlp_measure_fft_peak(0)
    print(r, flush=True)
    fma = 256 * 64 * 2.4e9  # double-precision FMAs per second at the peak clock
    # 6 FMAs forward and 8 operations inverse; the rest is left for a slower clock and latency.
    assert 0.6 * fma < 6 * r["fwd"] < 1.02 * fma, r
    assert 0.6 * fma < 8 * r["inv"] < 1.02 * fma, r
    assert r["inv"] <= r["mixed"] <= r["fwd"]


def test_bad_device_is_rejected():
    from paper_2506_12761_amd import vlp
    with pytest.raises(vlp.VlpError) as e:
        vlp.vlp_measure_fft_peak(4096)
    assert e.value.status == vlp.VLP_EINVAL
