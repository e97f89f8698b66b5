// Small disks (FFT size 64, boxes up to 32 x 32) resident on one CU.
//
// llg_resident: one workgroup of eight wavefronts owns a disk for the whole
// launch and keeps everything the step loop touches on chip: the row spectra
// and the stage state in LDS, the step's start state, the accumulator, the
// kernel spectra and the twiddles in registers.  Global memory is read at the
// start and written at the end, and there is no exchange between workgroups, so
// the launch needs neither group barriers nor co-residency.
//
// What bounds it: a lone small disk spread over several workgroups waits for
// two group barriers and the round trips through L2 in every stage (6.95 us a
// stage for R = 30 nm on 5 workgroups, 11.6 us on one workgroup of 192 threads);
// here a stage has two workgroup barriers and is bound by the vector issue of
// one CU.
//
// A stage's transforms (all of 64 points, 8 lanes x 8 points, two radix-8
// passes with one exchange through LDS):
// * rows: m_x + i m_y of every row as one complex transform F, and the two m_z
//   rows of a pair as another one, Q = FFT(m_z,2p + i m_z,2p+1): 32 + 16
//   transforms, six per wavefront, and neither is separated into the spectra of
//   the real rows.
// * columns: wavefronts 0-3 take F, 4-7 take Q, eight column pairs (kx, 64 - kx)
//   each.  With U = F(k) and V = conj F(-k) (the transform of the conjugated
//   column 64 - kx) the field spectrum is
//     H_x + i H_y = a U + (b + i K_xy) V,   a, b = (K_xx +- K_yy) / 2,
//   and its conjugate at -k is a V + (b - i K_xy) U: the pair needs no other
//   column.  A column of m_z is rebuilt from Q(kx) and conj Q(-kx) where it is
//   loaded: row 2p is their half sum, row 2p + 1 their half difference over i.
//   The self-paired columns kx = 0 and 32 share slot 0: for F they are its two
//   transforms, for m_z, whose columns 0 and 32 are real, one packed transform;
//   there K_xy = 0 and -k is the same column reversed.
// Wavefront w transforms the rows 4w .. 4w + 3 that its own threads update (a
// thread has the two cells of a row-pair column), so inverse transform, cell
// update and forward transform follow each other without a workgroup barrier.
#pragma once
#include "llg_device.hpp"

namespace llg {

constexpr int RES_P = 64;                  // FFT size
constexpr int RES_N = 32;                  // largest box
constexpr int RES_THREADS = 512;           // 8 wavefronts
constexpr int RES_ROW = 72;                // complex slots of a row buffer: 64 points, one pad after every 8
constexpr int RES_MW = 36;                 // floats of a staged row (columns -1 .. 34)

// One workgroup per CU: the step loop holds more registers than the 128 that two would leave each thread.
constexpr int RES_WAVES_PER_SIMD = 2;

struct ResLds {
    float2 S[(RES_N + RES_N / 2) * RES_ROW];             // rows 0..31: F or (H_x, H_y); 32..47: Q or (H_z, H_z) of a pair
    float2 X[(RES_THREADS / 8) * RES_ROW];               // exchange buffers of the column transforms
    float M[3][(RES_N + 2) * RES_MW];                    // stage state, one margin cell around the box
    double red[RES_THREADS / 64][4];                     // float64 sums per wavefront
};

// 64-point transform of the 8 lanes t of a group: on entry v[j] = x[t + 8 j], on
// exit v[j] = X[t + 8 j]; w[j] = exp(-2 pi i t j / 64).  LO: x[32 ..] is zero.
template <bool INV, bool LO>
__device__ __forceinline__ void fft64(float2 (&v)[8], float2* buf, const float2 (&w)[8], int t) {
    if constexpr (LO)
        dft8_lo<INV>(v);
    else
        dft8<INV>(v);
    wave_sync();
#pragma unroll
    for (int j = 0; j < 8; ++j) buf[9 * t + j] = v[j];
    wave_sync();
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = buf[t + 9 * j];
#pragma unroll
    for (int j = 1; j < 8; ++j) v[j] = INV ? cmulc(v[j], w[j]) : cmul(v[j], w[j]);
    dft8<INV>(v);
}

// conj X(-k) of the transform X held by the 8 lanes of a group (v[j] = X[t + 8 j])
__device__ __forceinline__ void conj_reversed(const float2 (&v)[8], float2 (&r)[8], int lane) {
    const int t = lane & 7, src = (lane & ~7) | ((8 - t) & 7);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float x = __shfl(v[7 - j].x, src, 64), y = __shfl(v[7 - j].y, src, 64);
        const float2 own = v[(8 - j) & 7];
        r[j] = t == 0 ? make_float2(own.x, -own.y) : make_float2(x, -y);
    }
}

__device__ __forceinline__ float lane_xor1(float x) {   // value of the neighbouring lane t ^ 1
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, true));
}

template <int MODE, bool SER>
__global__ __launch_bounds__(RES_THREADS) __attribute__((amdgpu_waves_per_eu(RES_WAVES_PER_SIMD)))
void llg_resident(KArgs a) {
    __shared__ ResLds L;
    const int k = blockIdx.x;
    const DiskDesc d = a.disks[k];
    const DiskPrm pr = a.prm[k];
    const int D = d.D, DD = D * D;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int slot = lane >> 3, t = lane & 7;
    const int mode = (MODE == MODE_DEMAG) ? a.mode : MODE;
    float* const m = a.m + d.m_off;

    // cells of this thread: column i of row pair p
    const int p = tid >> 5, i = tid & 31, j0 = 2 * p;
    const bool in[2] = {in_disk(j0, i, D), in_disk(j0 + 1, i, D)};   // false outside the box
    const int cell0 = j0 * D + i;

    // twiddles of this lane's transforms
    float2 w[8];
    twiddle_powers<8>(ldg2(d.tw + t), w);

    // kernel spectra of this lane's column points ky = t + 8 j
    const bool xy = wv < 4;                     // column work: F (m_x + i m_y) or Q (m_z)
    const int c = (wv & 3) * 8 + slot;          // column pair (c, 64 - c); c = 0: columns 0 and 32
    const int c2 = c ? RES_P - c : RES_P / 2;
    float ka[8], kb[8], kc[8], kd[8];
    {
        constexpr int H = RES_P / 2 + 1;
        const GLOBAL_AS float* sp = gbl(d.spec);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int ky = t + 8 * j, kq = ky <= 32 ? ky : 64 - ky;
            auto at = [&](int plane, int kx) { return sp[(plane * H + kx) * H + kq]; };
            kb[j] = kc[j] = kd[j] = 0.f;
            if (xy) {
                const float xx = at(0, c), yy = at(1, c);
                ka[j] = 0.5f * (xx + yy);
                kb[j] = 0.5f * (xx - yy);
                if (c) {
                    kc[j] = ky <= 32 ? at(2, c) : -at(2, c);   // K_xy is odd in ky
                } else {
                    const float x2 = at(0, 32), y2 = at(1, 32);
                    kc[j] = 0.5f * (x2 + y2);
                    kd[j] = 0.5f * (x2 - y2);
                }
            } else {
                ka[j] = 0.5f * at(3, c);
                if (!c) {
                    const float z2 = 0.5f * at(3, 32);
                    kd[j] = ka[j] - z2;
                    ka[j] += z2;
                }
            }
        }
    }

    // ---- state of the two cells, into registers and the row buffers
    float cur[2][3], base[2][3], acc[2][3];
    float2* const own0 = &L.S[j0 * RES_ROW + padb(i)];                  // (x, y) of row j0; row j0 + 1 follows
    float2* const ownz = &L.S[(RES_N + p) * RES_ROW + padb(i)];         // the pair's (z, z)
    auto store_rows = [&](const float (&v)[2][3]) {
        own0[0] = make_float2(v[0][0], v[0][1]);
        own0[RES_ROW] = make_float2(v[1][0], v[1][1]);
        ownz[0] = make_float2(v[0][2], v[1][2]);
    };
    float* const stage = &L.M[0][(j0 + 1) * RES_MW + i + 1];            // this thread's staged cells
    constexpr int PL = (RES_N + 2) * RES_MW;
    auto stage_cells = [&]() {
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int q = 0; q < 3; ++q) stage[q * PL + r * RES_MW] = cur[r][q];
    };
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            cur[r][q] = in[r] ? gbl(m)[q * DD + cell0 + r * D] : 0.f;
            base[r][q] = acc[r][q] = 0.f;
        }
    for (int e = tid; e < 3 * PL; e += RES_THREADS) (&L.M[0][0])[e] = 0.f;   // the margins stay zero

    // ---- row transforms of this wavefront: rows 4 wv .. + 3 in slots 0 .. 3, pairs 2 wv, 2 wv + 1 in slots 4, 5
    float2* const rowb = &L.S[(slot < 4 ? 4 * wv + slot : RES_N + 2 * wv + (slot & 1)) * RES_ROW];
    auto rows_forward = [&]() {
        wave_sync();
        if (slot < 6) {
            float2 v[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = rowb[t + 9 * j];
            fft64<false, true>(v, rowb, w, t);
            wave_sync();
#pragma unroll
            for (int j = 0; j < 8; ++j) rowb[t + 9 * j] = v[j];
        }
    };
    auto rows_inverse = [&]() {
        if (slot < 6) {
            float2 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = rowb[t + 9 * j];
            fft64<true, false>(v, rowb, w, t);
            wave_sync();
#pragma unroll
            for (int j = 0; j < 4; ++j) rowb[t + 9 * j] = v[j];
        }
        wave_sync();
    };

    // ---- column transforms and the spectral product
    float2* const xb = &L.X[(tid >> 3) * RES_ROW];
    auto columns = [&]() {
        float2* const colA = &L.S[padb(c)];
        float2* const colB = &L.S[padb(c2)];
        if (xy) {
            float2 U[8], V[8];
            const float sg = c ? -1.f : 1.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                U[j] = colA[(t + 8 * j) * RES_ROW];
                V[j] = colB[(t + 8 * j) * RES_ROW];
                V[j].y *= sg;
            }
            fft64<false, true>(U, xb, w, t);
            fft64<false, true>(V, xb, w, t);
            if (wv == 0) {   // slot 0: U' = a U + b conj U(-), V' = kc V + kd conj V(-)
                float2 ur[8], vr[8];
                conj_reversed(U, ur, lane);
                conj_reversed(V, vr, lane);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float2 u = U[j], v = V[j];
                    const float2 g = make_float2(ka[j] * u.x + (kb[j] * v.x - kc[j] * v.y),
                                                 ka[j] * u.y + (kb[j] * v.y + kc[j] * v.x));
                    const float2 h = make_float2(ka[j] * v.x + (kb[j] * u.x + kc[j] * u.y),
                                                 ka[j] * v.y + (kb[j] * u.y - kc[j] * u.x));
                    U[j] = c ? g : make_float2(ka[j] * u.x + kb[j] * ur[j].x, ka[j] * u.y + kb[j] * ur[j].y);
                    V[j] = c ? h : make_float2(kc[j] * v.x + kd[j] * vr[j].x, kc[j] * v.y + kd[j] * vr[j].y);
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float2 u = U[j], v = V[j];
                    U[j] = make_float2(ka[j] * u.x + (kb[j] * v.x - kc[j] * v.y),
                                       ka[j] * u.y + (kb[j] * v.y + kc[j] * v.x));
                    V[j] = make_float2(ka[j] * v.x + (kb[j] * u.x + kc[j] * u.y),
                                       ka[j] * v.y + (kb[j] * u.y - kc[j] * u.x));
                }
            }
            fft64<true, false>(U, xb, w, t);
            fft64<true, false>(V, xb, w, t);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                colA[(t + 8 * j) * RES_ROW] = U[j];
                colB[(t + 8 * j) * RES_ROW] = make_float2(V[j].x, sg * V[j].y);
            }
        } else {
            // rows t + 8 j = 2 (t / 2 + 4 j) + (t & 1): even lanes take the half sum, odd ones the half difference
            // (the halves are in ka)
            float2 z[8];
            const bool odd = t & 1;
            const int q0 = (RES_N + (t >> 1)) * RES_ROW;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2 A = colA[q0 + 4 * j * RES_ROW], B = colB[q0 + 4 * j * RES_ROW];
                // A + conj B, and (A - conj B) / i
                const float2 e = make_float2(A.x + B.x, A.y - B.y), o = make_float2(A.y + B.y, B.x - A.x);
                const float2 e0 = make_float2(A.x, B.x), o0 = make_float2(A.y, B.y);
                z[j] = c ? (odd ? o : e) : (odd ? o0 : e0);
            }
            fft64<false, true>(z, xb, w, t);
            if (wv == 4) {
                float2 zr[8];
                conj_reversed(z, zr, lane);
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    z[j] = make_float2(ka[j] * z[j].x + kd[j] * zr[j].x, ka[j] * z[j].y + kd[j] * zr[j].y);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) z[j] = make_float2(ka[j] * z[j].x, ka[j] * z[j].y);
            }
            fft64<true, false>(z, xb, w, t);
            // Q(c) = z_2p + i z_2p+1 from the even lane, Q(-c) = conj z_2p + i conj z_2p+1 from the odd one
            float2* const to = odd ? colB : colA;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2 n = make_float2(lane_xor1(z[j].x), lane_xor1(z[j].y));
                const float2 e = odd ? n : z[j], o = odd ? z[j] : n;      // rows 2p and 2p + 1
                const float2 gen = odd ? make_float2(e.x + o.y, o.x - e.y) : make_float2(e.x - o.y, e.y + o.x);
                const float2 sp0 = odd ? make_float2(e.y, o.y) : make_float2(e.x, o.x);
                to[q0 + 4 * j * RES_ROW] = c ? gen : sp0;
            }
        }
    };

    // ---- external field of the stage
    float hxf = pr.hx, hyf = pr.hy, hzf = pr.hz;
    double hxd = pr.hx_d, hyd = pr.hy_d, hzd = pr.hz_d;
    auto set_field = [&](double tau) {
        if (pr.drive) {
            if constexpr (MODE == MODE_RK4 || MODE == MODE_HEUN) {
                hext_at_f(pr, tau, hxf, hyf, hzf);
                hxd = hxf;
                hyd = hyf;
                hzd = hzf;
            } else {
                const Field3 h = hext_at(pr, tau);
                hxd = h.x;
                hyd = h.y;
                hzd = h.z;
                hxf = (float)h.x;
                hyf = (float)h.y;
                hzf = (float)h.z;
            }
        }
    };

    // float64 sums over the disk of q4 (NQ values): every wavefront's into LDS; thread q < NQ
    // returns the total of value q after the caller's workgroup barrier
    auto wave_sums = [&](const double* q4, int nq) {
        for (int q = 0; q < nq; ++q) {
            const double v = wave_sum(q4[q]);
            if (lane == 0) L.red[wv][q] = v;
        }
    };
    auto total = [&](int q) {
        double v = 0.0;
        for (int g = 0; g < RES_THREADS / 64; ++g) v += L.red[g][q];
        return v;
    };

    const float cf = pr.c, al = pr.alpha, dt = pr.dtau;
    constexpr int NST = (MODE == MODE_HEUN) ? 2 : 4;
    float* const recd = a.rec ? a.rec + (size_t)a.nsteps * (2 * NST) * (size_t)d.m_off : nullptr;
    const unsigned long long step0 = (MODE == MODE_HEUN && a.step_ptr) ? *gbl(a.step_ptr) : a.step0;
    // neighbour sums of the two cells (exchange), in the order row above, row below, left, right
    auto neighbours = [&](int r, int q) {
        const float* s = stage + q * PL + r * RES_MW;
        const float up = r == 0 ? s[-RES_MW] : cur[0][q], dn = r == 0 ? cur[1][q] : s[RES_MW];
        return make_float4(up, dn, s[-1], s[1]);
    };

    store_rows(cur);
    rows_forward();
    __syncthreads();

    if constexpr (MODE == MODE_DEMAG) {
        set_field(pr.tau0);
        stage_cells();
        columns();
        __syncthreads();
        rows_inverse();
        float* const out = a.out ? a.out + d.m_off : nullptr;
        double e3[3] = {0.0, 0.0, 0.0};
        const float2 hz2 = ownz[0];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const float2 hxy = own0[r * RES_ROW];
            const float H[3] = {hxy.x, hxy.y, r == 0 ? hz2.x : hz2.y};
            const bool box = i < D && j0 + r < D;
            float res[3] = {H[0], H[1], H[2]};
            if (mode == MODE_ENERGY) {
                if (!in[r]) continue;
                const double h3[3] = {hxd, hyd, hzd};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float4 nb = neighbours(r, q);
                    const double mq = cur[r][q];
                    e3[0] += -0.5 * mq * ((double)nb.x + (double)nb.y + (double)nb.z + (double)nb.w);
                    e3[1] += -0.5 * pr.c_d * mq * (double)H[q];
                    e3[2] += -pr.c_d * mq * h3[q];
                }
                continue;
            }
            if (mode == MODE_RHS) {
                float b[3];
                const float h3[3] = {hxf, hyf, hzf};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float4 nb = neighbours(r, q);
                    b[q] = (nb.x + nb.y + nb.z + nb.w) + cf * (h3[q] + H[q]);
                }
                const float mx = cur[r][0], my = cur[r][1], mz = cur[r][2];
                const float px = my * b[2] - mz * b[1], py = mz * b[0] - mx * b[2], pz = mx * b[1] - my * b[0];
                res[0] = px - al * (my * pz - mz * py);
                res[1] = py - al * (mz * px - mx * pz);
                res[2] = pz - al * (mx * py - my * px);
            }
            if (box)
#pragma unroll
                for (int q = 0; q < 3; ++q) gbl(out)[q * DD + cell0 + r * D] = in[r] ? res[q] : 0.f;
        }
        if (mode == MODE_ENERGY) {
            wave_sums(e3, 3);
            __syncthreads();
            if (tid < 3) gbl(a.part)[k * PART_STRIDE + tid] = total(tid);
        }
    } else {
        for (long long n = 0; n < a.nsteps; ++n) {
#pragma unroll 1
            for (int s = 0; s < NST; ++s) {
                stage_cells();   // the stencil of the stage before is done (workgroup barrier)
                columns();
                __syncthreads();
                const double frac = NST == 4 ? (s == 0 ? 0.0 : s == 3 ? 1.0 : 0.5) : (double)s;
                set_field(pr.tau0 + ((double)n + frac) * pr.dtau_d);
                rows_inverse();
                const bool last = n == a.nsteps - 1 && s == NST - 1;
                const bool sampled = SER && s == 0 && n % a.every == 0;
                double q4[4] = {0.0, 0.0, 0.0, 0.0};
                const float2 hz2 = ownz[0];
                float3 wn[2];
                if (MODE == MODE_HEUN && (in[0] || in[1]))
                    thermal_normals_pair(a.seed, step0 + (unsigned long long)n, (unsigned long long)(p * D + i),
                                         (unsigned long long)(a.replica0 + d.k), wn[0], wn[1]);
                float nxt[2][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const float2 hxy = own0[r * RES_ROW];
                    const float H[3] = {hxy.x, hxy.y, r == 0 ? hz2.x : hz2.y};
                    if (!in[r]) {
                        if (recd && i < D && j0 + r < D) {
                            GLOBAL_AS float* rs = gbl(recd) + ((size_t)(n * NST + s) * 2) * 3 * DD + cell0 + r * D;
#pragma unroll
                            for (int q = 0; q < 6; ++q) rs[q * DD] = 0.f;
                        }
                        continue;
                    }
                    const float h3[3] = {hxf, hyf, hzf};
                    float b[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const float4 nb = neighbours(r, q);
                        b[q] = (nb.x + nb.y + nb.z + nb.w) + cf * (h3[q] + H[q]);
                        if (SER && sampled) {
                            const double hd[3] = {hxd, hyd, hzd};
                            const double mq = cur[r][q];
                            q4[q] += mq;
                            q4[3] += -0.5 * mq * ((double)nb.x + (double)nb.y + (double)nb.z + (double)nb.w) -
                                     pr.c_d * mq * (hd[q] + 0.5 * (double)H[q]);
                        }
                    }
                    const float mx = cur[r][0], my = cur[r][1], mz = cur[r][2];
                    if (recd) {
                        GLOBAL_AS float* rs = gbl(recd) + ((size_t)(n * NST + s) * 2) * 3 * DD + cell0 + r * D;
#pragma unroll
                        for (int q = 0; q < 3; ++q) {
                            rs[q * DD] = cur[r][q];
                            rs[(3 + q) * DD] = H[q];
                        }
                    }
                    if constexpr (MODE == MODE_HEUN) {   // g = b dtau + sigma w
                        const float3 wr = wn[r];
                        b[0] = b[0] * dt + pr.sigma * wr.x;
                        b[1] = b[1] * dt + pr.sigma * wr.y;
                        b[2] = b[2] * dt + pr.sigma * wr.z;
                    }
                    // f = m x b - alpha m x (m x b)
                    const float px = my * b[2] - mz * b[1], py = mz * b[0] - mx * b[2], pz = mx * b[1] - my * b[0];
                    const float f[3] = {px - al * (my * pz - mz * py), py - al * (mz * px - mx * pz),
                                        pz - al * (mx * py - my * px)};
                    bool done = false;
                    if constexpr (MODE == MODE_RK4) {
                        if (s < 3) {
                            const float h = (s == 2) ? dt : 0.5f * dt, wgt = (s == 0) ? 1.f : 2.f;
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                if (s == 0) base[r][q] = cur[r][q];
                                acc[r][q] = (s == 0 ? 0.f : acc[r][q]) + wgt * f[q];
                                nxt[r][q] = base[r][q] + h * f[q];
                            }
                        } else {
                            const float h6 = dt * (1.0f / 6.0f);
#pragma unroll
                            for (int q = 0; q < 3; ++q) nxt[r][q] = base[r][q] + h6 * (acc[r][q] + f[q]);
                            done = true;
                        }
                    } else {
                        if (s == 0) {   // predictor; m + Delta_1 / 2 kept for the corrector
#pragma unroll
                            for (int q = 0; q < 3; ++q) {
                                acc[r][q] = cur[r][q] + 0.5f * f[q];
                                nxt[r][q] = cur[r][q] + f[q];
                            }
                        } else {
#pragma unroll
                            for (int q = 0; q < 3; ++q) nxt[r][q] = acc[r][q] + 0.5f * f[q];
                            done = true;
                        }
                    }
                    if (done) {
                        float x = nxt[r][0], y = nxt[r][1], z = nxt[r][2];
                        if (pr.renorm) {
                            const float rn = 1.0f / sqrtf(x * x + y * y + z * z);
                            x *= rn;
                            y *= rn;
                            z *= rn;
                        }
                        if (!(isfinite(x) && isfinite(y) && isfinite(z))) raise_err(a.err, (int)ERR_NONFINITE);
                        nxt[r][0] = x;
                        nxt[r][1] = y;
                        nxt[r][2] = z;
                    }
                }
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int q = 0; q < 3; ++q) cur[r][q] = nxt[r][q];
                if (SER && sampled) wave_sums(q4, 4);
                if (!last) {
                    store_rows(cur);
                    rows_forward();
                }
                __syncthreads();
                if (SER && sampled && tid < 4) {   // red is next written after further workgroup barriers
                    const double v = total(tid);
                    gbl(a.series)[((n / a.every) * a.n_disks + d.k) * 4 + tid] = tid < 3 ? v / (double)d.n_cells : v;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if (i < D && j0 + r < D)
#pragma unroll
                for (int q = 0; q < 3; ++q) gbl(m)[q * DD + cell0 + r * D] = cur[r][q];
    }
}

}  // namespace llg
