/* Host build of the device math header (plain C): lets the CPU tests compare the exact
 * functions the kernels use with libm, value by value. */
#include "q8_math.h"

void q8m_tanh(const float *x, float *y, long n) { for (long i = 0; i < n; ++i) y[i] = q8_tanh_rn(x[i]); }
void q8m_sigmoid(const float *x, float *y, long n) { for (long i = 0; i < n; ++i) y[i] = q8_sigmoid_rn(x[i]); }
void q8m_exp(const double *x, double *y, long n) { for (long i = 0; i < n; ++i) y[i] = q8_exp_d(x[i]); }

/* tanh of the sums p[i] + a[i], four at a time (n % 4 == 0) */
void q8m_tanh_sums(const float *p, const float *a, float *y, long n)
{
    for (long i = 0; i < n; i += 4) {
        double ep[4], ea[4];
        for (int c = 0; c < 4; ++c) {
            ep[c] = 2.0 * q8_exp_d(2.0 * (double)p[i + c]);
            ea[c] = q8_exp_d(2.0 * (double)a[i + c]);
        }
        q8_tanh4_sums(p + i, a + i, ep, ea, y + i);
    }
}
