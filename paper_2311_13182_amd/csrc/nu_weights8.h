// Generated by gen_nu_weights.py (do not edit): least-squares polynomial
// forms of the 8 tap weights of the exponential-of-semicircle kernel of width
// 8, beta = 18.40, in the offset u in [-1/2, 1/2] from the middle between two
// grid points: w_t = E_t(u^2) + u O_t(u^2), w_{7-t} = E_t(u^2) - u O_t(u^2)
// (t < 4); coefficients by ascending power of u^2.  Largest deviation from
// the kernel on the fitting grid: 9.01e-08.
#pragma once

constexpr int kNu8PolyNE = 4, kNu8PolyNO = 4;   // coefficients per polynomial
constexpr float kNu8PolyE[4][4] = {
    {7.544830751e-05f, 2.224266900e-03f, 5.317514617e-03f, 1.366037719e-03f},
    {1.765907471e-02f, 9.842144320e-02f, 2.131586195e-02f, -7.217366994e-03f},
    {2.611283060e-01f, 2.636088612e-01f, -9.573844124e-02f, 1.321612541e-02f},
    {8.656142004e-01f, -3.642560096e-01f, 6.911543708e-02f, -7.388415241e-03f}
};
constexpr float kNu8PolyO[4][4] = {
    {-6.272385825e-04f, -4.403745550e-03f, -3.884115827e-03f, 3.805329101e-05f},
    {-6.503747194e-02f, -7.388939996e-02f, 7.444343686e-03f, 1.109728892e-03f},
    {-4.859053895e-01f, 4.973947696e-02f, 1.650722478e-02f, -4.649459771e-03f},
    {-5.016627483e-01f, 2.510846758e-01f, -5.972514642e-02f, 8.540967657e-03f}
};
