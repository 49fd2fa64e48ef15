// Host packing of inputs: the caller's FP64 hits, states and covariances into
// the FP32 forms the kernels read, with their checks.  Plain C++, compiled for
// the widest vectors the host has: a hit costs a square root and two
// divisions in FP64, eight hits at a time instead of one (500 seeds and 6,500
// hits on one thread: 8 us, one value at a time 21).  Built without fused
// multiply-adds, so that every width rounds as the scalar form does.
#include "mkf_pack.hpp"

#include <cmath>

namespace mkf {

namespace {

constexpr double kPiD = 3.14159265358979323846;

inline __attribute__((always_inline)) bool narrow_body(const double *__restrict src, float *__restrict dst, size_t n)
{
    int bad = 0;
    for (size_t i = 0; i < n; ++i) {
        const float f = (float)src[i];
        dst[i] = f;
        bad |= !(f - f == 0.f);   // infinite or NaN
    }
    return bad == 0;
}

template <HitForm kForm>
inline __attribute__((always_inline)) bool hits_body(const double *__restrict h, size_t n, float *__restrict out)
{
    int bad = 0;
    for (size_t i = 0; i < n; ++i) {
        const double x = h[3 * i], y = h[3 * i + 1], z = h[3 * i + 2];
        const double r = std::sqrt(x * x + y * y);
        float a, b, c, d;
        if (kForm == HitForm::kXyz) {
            a = (float)x, b = (float)y, c = (float)z, d = 0.f;
            bad |= !((double)a * a + (double)b * b > 0);
        } else {
            a = (float)(x / r), b = (float)(y / r);
            c = (float)(kForm == HitForm::kDisk ? r : z);
            d = (float)(kForm == HitForm::kDisk ? z : r);
        }
        bad |= !(r > 0) | !(a - a == 0.f) | !(b - b == 0.f) | !(c - c == 0.f) | !(d - d == 0.f);
        out[4 * i] = a, out[4 * i + 1] = b, out[4 * i + 2] = c, out[4 * i + 3] = d;
    }
    return bad == 0;
}

inline __attribute__((always_inline)) bool states_body(const double *__restrict par, size_t n)
{
    int bad = 0;
    for (size_t i = 0; i < n; ++i) {
        const double *p = par + 6 * i;
        bad |= !(p[5] > 0) | !(p[5] < kPiD) | !(p[0] * p[0] + p[1] * p[1] > 0);
    }
    return bad == 0;
}

#define MKF_WIDTHS(X) X(avx512, "avx512f,avx512dq,avx512vl,avx512bw") X(avx2, "avx2")
#define MKF_DEFINE(name, features)                                                                              \
    __attribute__((target(features))) bool narrow_##name(const double *s, float *d, size_t n)                  \
    {                                                                                                          \
        return narrow_body(s, d, n);                                                                           \
    }                                                                                                          \
    template <HitForm kForm>                                                                                   \
    __attribute__((target(features))) bool hits_##name(const double *h, size_t n, float *o)                    \
    {                                                                                                          \
        return hits_body<kForm>(h, n, o);                                                                      \
    }                                                                                                          \
    __attribute__((target(features))) bool states_##name(const double *p, size_t n) { return states_body(p, n); }
MKF_WIDTHS(MKF_DEFINE)

int host_width()
{
    static const int w = __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512dq") &&
                                 __builtin_cpu_supports("avx512vl") && __builtin_cpu_supports("avx512bw")
                             ? 2
                             : __builtin_cpu_supports("avx2") ? 1 : 0;
    return w;
}

template <HitForm kForm>
bool hits_of(const double *h, size_t n, float *o)
{
    const int w = host_width();
    return w == 2 ? hits_avx512<kForm>(h, n, o) : w == 1 ? hits_avx2<kForm>(h, n, o) : hits_body<kForm>(h, n, o);
}

}  // namespace

bool narrow_all(const double *src, float *dst, size_t n)
{
    const int w = host_width();
    return w == 2 ? narrow_avx512(src, dst, n) : w == 1 ? narrow_avx2(src, dst, n) : narrow_body(src, dst, n);
}

bool pack_hits(const double *h, size_t n, HitForm form, float *out)
{
    switch (form) {
    case HitForm::kXyz: return hits_of<HitForm::kXyz>(h, n, out);
    case HitForm::kDisk: return hits_of<HitForm::kDisk>(h, n, out);
    default: return hits_of<HitForm::kCylinder>(h, n, out);
    }
}

bool states_in_range(const double *par, size_t n)
{
    const int w = host_width();
    return w == 2 ? states_avx512(par, n) : w == 1 ? states_avx2(par, n) : states_body(par, n);
}

}  // namespace mkf
