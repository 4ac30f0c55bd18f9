"""Occupation rows (a group of strings that differ from a base in one qubit,
summed over the occupied qubits instead of term by term) are as accurate as
the terms they stand for: over random samples, the rms error of a group's sum
is at most 1.1 times that of its terms added in order (1.1: the spread of a
ratio of rms values over 2,000 sums), whatever the signs and sizes of the
coefficients.  The device function runs on the CPU as plain C++."""
from test_host_register import check

BODY = r"""
// kind 0: random signs; 1: one sign; 2: equal; 3: one sign, and a string
// without another qubit that balances them (the molecular form)
static void run(int nq, int kind) {
    const int groups = 10;
    std::vector<uint64_t> x, z;
    std::vector<double> c;
    for (int g = 0; g < groups; ++g) {
        double sum = 0.0;
        const uint64_t X = 5ull << g;
        for (int q = 0; q < nq; ++q) {
            if ((X >> q) & 1) continue;
            const double v = kind == 0 ? uniform() : kind == 2 ? 1.0 / 3.0 : 0.25 + uniform() * uniform();
            x.push_back(X); x.push_back(0);
            z.push_back(1ull << q); z.push_back(0);
            c.push_back(v);
            sum += v;
        }
        if (kind == 3) {
            x.push_back(X); x.push_back(0);
            z.push_back(0); z.push_back(0);
            c.push_back(-sum);
        }
    }
    HostTable T;
    std::string err;
    if (build_table(nq, static_cast<int64_t>(c.size()), x.data(), z.data(), c.data(), nullptr, &T, &err)) {
        ++bad;
        return;
    }
    GroupRecords R;
    build_group_records(T, &R);
    std::vector<uint32_t> goff(T.goff.begin(), T.goff.end());
    DevTable tab{};
    tab.n_qubits = nq;
    tab.gx = R.rec.data();
    tab.gx_stride = kGroupWords;
    tab.goff = goff.data();
    tab.tz = R.z.data();
    tab.tc = T.tc.data();
    tab.tcode = R.codes.data();
    tab.occ = R.rows.data();
    double by_group = 0.0, by_terms = 0.0;
    unsigned long long terms = 0;
    for (int k = 0; k < 2000; ++k) {
        const Key<1> s = sample<1>(nq, 0);
        const int64_t g = k % groups;
        double t = 0.0;
        long double exact = 0.0L;
        for (int64_t i = T.goff[g]; i < T.goff[g + 1]; ++i) {
            const double v = __builtin_parityll(T.tz[2 * i] & s.w[0]) ? -T.tc[i] : T.tc[i];
            t += v;
            exact += v;
        }
        const double a = static_cast<double>(group_sum<1, false>(tab, g, s, nullptr, &terms) - exact);
        const double b = static_cast<double>(t - exact);
        by_group += a * a;
        by_terms += b * b;
    }
    const double ratio = std::sqrt(by_group / by_terms);
    std::printf("%d qubits, kind %d: %d rows, rms ratio %.2f\n", nq, kind,
                static_cast<int>(R.rows.size()), ratio);
    expect(ratio <= 1.1, "error above the terms'", nq);
    if (kind == 3) expect(!R.rows.empty(), "rows where they are as accurate", nq);
}
int main() {
    for (int kind = 0; kind < 4; ++kind) { run(24, kind); run(40, kind); run(62, kind); }
    return bad != 0;
}
"""


def test_rows_are_as_accurate_as_their_terms(tmp_path):
    check(tmp_path, BODY)
