"""The profile summaries' kernel names and element counts (CPU): every kernel that
the benchmark's workloads launch is named by what it evaluates."""
from paper_2605_15547_amd import rocpd_summary as R

NS = "(anonymous namespace)::"


def test_kernel_names():
    for name, want in (
            ("void %sk_map_f32<%sOpLog<3>, 2, 1, 0>(float const*)", "k_map_f32<OpLog<3>> (log1pf)"),
            ("void %sk_tiles<%sBOne<%sOpSTrig<0> > >(int)", "k_tiles<OpSTrig<0>> (sinf split)"),
            ("void %sk_dft<false>(float const*, int)", "k_dft<false> (dft)"),
            ("void %sk_dft<true>(float const*, int)", "k_dft<true> (dft, one slice)"),
            ("void %sk_batch<true>(int)", "k_batch<true> (batch split)"),
            ("void %sk_batch_args<false>(int)", "k_batch_args<false> (batch)")):
        assert R.short(name.replace("%s", NS)) == want


def test_the_dft_counts_its_terms():
    n = R.elems_of(R.short("void " + NS + "k_dft<false>(float const*, int)"), {})
    assert n == (1 << 20) * 256
    assert R.elems_of("k_dft_finish", {}) is None
