"""The reads of the coarse tail's restriction stay inside the finer level's residuals
(no GPU): the index arithmetic of np_tail.hip, compiled for the host, over every pair
of levels a plan may hold and every slot of the coarse level, among them the one past
an odd N_x that holds no point."""
from hip_stub import run_host_part

CODE = r"""
#include <cstdio>
// N: points of a coarse level along an axis, F: of the finer one (2 N <= F + 1, F / 2 <= N)
template <int D>
int check(int n)
{
    for (int m = 0; m < 3 * 3 * (D == 3 ? 3 : 1); m++) {
        const int F[3] = {2 * n - 1 + m % 3, 2 * (n + 1) - 1 + m / 3 % 3, D == 3 ? 2 * (n + 2) - 1 + m / 9 : 1};
        const int slots = 2 * ((n + 1) / 2), total = F[0] * F[1] * F[2];
        for (int k = 1; k <= (D == 3 ? n + 2 : 1); k++)
            for (int j = 1; j <= n + 1; j++)
                for (int i = 1; i <= slots; i++) {
                    const auto q = np::tail_kids<D>(i, j, D == 3 ? k : 0, n, F);
                    const int end = q.at + q.dx + q.dy + q.dz;
                    if (q.at < 0 || end >= total) {
                        printf("%d-D, N = %d, F = %d %d %d: point %d %d %d reads %d .. %d of %d\n", D, n, F[0], F[1], F[2], i, j, k,
                               q.at, end, total);
                        return 1;
                    }
                    // a point's own children: each inside one once
                    if (i <= n && (q.inx != (2 * i <= F[0]) || q.iny != (2 * j <= F[1]) || (D == 3 && q.inz != (2 * k <= F[2])) ||
                                   q.at != ((D == 3 ? 2 * k - 2 : 0) * F[1] + 2 * j - 2) * F[0] + 2 * i - 2))
                        return 2;
                }
    }
    return 0;
}
int main()
{
    for (int n = 1; n <= 20; n++)
        if (check<2>(n) || check<3>(n)) return 1;
    return 0;
}
"""


def test_restriction_reads_inside(tmp_path):
    run_host_part("np_tail.hip", CODE, str(tmp_path))
