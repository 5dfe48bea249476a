// direct.hpp -- the direct-load variants of the macro-kernel (device code).
//
// When both operands are gathered in 16-byte vectors (row or k vectors; on
// the Y side also k vectors strided by the split of the K box),
// packing (Eq. 9-10) needs no registers: the load unit copies each 16-byte
// piece from device memory straight into LDS (global_load_lds_dwordx4: lane
// i of one instruction fills bytes [16 i, 16 i + 16) after a wave-uniform LDS
// base); a piece outside the tensors is written as zeros by its thread.
// The LDS layout of an operand tile is then fixed by which piece each lane
// loads:
//   row-vector operand: [k][row], as the macro-kernel packs it (no padding);
//   k-vector operand:   [row][k], the pieces of row r XOR-permuted by
//                       (r / R) mod (pieces per row) -- rotated by r / R when
//                       the pieces per row are not a power of two -- so that
//                       the lanes of an MFMA read, which take rows R apart at
//                       one k piece (R = 4 in fp32, 2 in fp64), fall on
//                       different banks.
//   strided k-vector:   [row][k] likewise; a piece holds VW positions es apart,
//                       so the MFMA steps read it element by element.
// A k-vector piece holds VW consecutive contracted positions, and one LDS
// read hands them to VW consecutive MFMA steps: the position lane group g
// supplies in step s is
//   kp(s, g) = 4 VW floor(s / VW) + VW g + (s mod VW)
// on both operands (a bijection of the box's KT positions onto the (s, g)
// pairs, so each product still pairs matching indices and the sum is the
// same up to rounding order).
//
// Pipeline, two LDS buffers, box s in buffer s mod 2:
//   MFMAs of box s's first step groups, from registers;
//   wait for this wavefront's loads of box s + 1; barrier (all loads of box
//     s + 1 have landed, every wavefront is done reading box s);
//   loads of box s + 2 into box s's buffer;
//   LDS reads of box s + 1's fragments, interleaved with the MFMAs of box s's
//     last step group.
// Nothing is staged in registers but the fragments, so a workgroup of eight
// wavefronts (two per SIMD) fits a 256 x 128 fp32 tile.
//
// The persistent variant (gett_direct_stream_kernel, contracted sets of one
// box) walks several tiles per workgroup and copies the next tile's box into
// the other buffer before storing the current tile's C, so the copy is not
// queued behind those stores.
#pragma once
#include "kernel.hpp"

namespace gett {

typedef __attribute__((address_space(1))) void global_void;
typedef __attribute__((address_space(3))) void lds_void;

// k-vector layout: LDS column of piece c of row r (CPR pieces per row, rows
// read R at a time).  With 2^n pieces per row the pieces are XOR-permuted by
// (r / R) mod CPR (an involution); otherwise rotated by r / R.
template <int CPR, int R>
__device__ __forceinline__ int kvec_col(int r, int c)
{
    if constexpr ((CPR & (CPR - 1)) == 0) return c ^ ((r / R) & (CPR - 1));
    else return (c + r / R) % CPR;
}
// the piece of row r held in LDS column c
template <int CPR, int R>
__device__ __forceinline__ int kvec_piece(int r, int c)
{
    if constexpr ((CPR & (CPR - 1)) == 0) return c ^ ((r / R) & (CPR - 1));
    else return (c + CPR - (r / R) % CPR) % CPR;
}

// The pieces of one operand tile (ROWS x KT elements) one thread loads per
// box: J per thread, piece p = (j * NW + wave) * 64 + lane of the tile's LDS
// image.  A piece outside the tensor (its rows past the tile's last, or its
// contracted positions past the box's valid ones) is not loaded: the thread
// writes zeros to its place instead, as the macro-kernel's gathers do.
// WHOLE: every box is whole (no checks; rows past the tile's last load its
// first row, and nothing reads their results).  R: rows one lane
// reads together from the [row][k] layout (RX / RY), which sets the row
// period of the k-vector permutation.
template <typename T, int ROWS, int KT, int MODE, int NTH, bool WHOLE, int R>
struct DirectOperand {
    static constexpr int VW = Traits<T>::VW;
    static constexpr int NW = NTH / 64;
    static constexpr int PIECES = ROWS * KT / VW;
    static constexpr int J = PIECES / NTH;
    static constexpr int CPR = KT / VW;     // k-vector layout: pieces per row
    static constexpr int RPL = ROWS / VW;   // row-vector layout: pieces per line
    static_assert(MODE == kGatherRowVec || MODE == kGatherKVec || MODE == kGatherKVecStrided,
                  "vector gathers only");
    static_assert(PIECES % NTH == 0 && J >= 1, "whole pieces per thread");
    static_assert(ROWS % VW == 0 && KT % VW == 0, "whole vectors");
    typedef typename Traits<T>::vec vec;

    int goff[J];               // element offset of each piece (tile base and box origin excluded)
    int kc[WHOLE ? 1 : J];     // position along index kj of its first element; kInvalidK: never valid
    int lane;

    // piece of row r held in LDS column c of the k-vector layout (the inverse
    // of kvec_col)
    static __device__ __forceinline__ int swz(int r, int c) { return kvec_piece<CPR, R>(r, c); }

    // rowoff: LDS table of operand offsets per tile row (-1 = outside the
    // tensor); koff / kco: offsets / kj-positions per box position; es: box
    // positions between the elements of a strided k-vector
    __device__ __forceinline__ void setup(int tid, const int *rowoff, const int *koff,
                                          const int *kco, int es = 1)
    {
        lane = tid & 63;
        const int w = tid >> 6;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int p = (j * NW + w) * 64 + lane;
            int r, kk;
            if constexpr (MODE == kGatherKVec) {
                r = p / CPR;
                kk = VW * swz(r, p % CPR);
            } else if constexpr (MODE == kGatherKVecStrided) {
                r = p / CPR;
                const int c = swz(r, p % CPR), nq = CPR / es;   // piece c: value c / nq of the
                kk = c / nq + (c % nq) * VW * es;               // first index, vector c % nq
            } else {
                r = VW * (p % RPL);
                kk = p / RPL;
            }
            const int ro = rowoff[r];
            goff[j] = (ro < 0 ? 0 : ro) + koff[kk];
            if constexpr (!WHOLE) kc[j] = ro < 0 ? kInvalidK : kco[kk];
        }
    }

    // copy this thread's pieces of the box at `base` (`lim` valid positions
    // along index kj) into the tile image `dst`
    __device__ __forceinline__ void issue(const T *base, T *dst, int w, int lim) const
    {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            T *slot = dst + (j * NW + w) * 64 * VW;
            if (WHOLE || kc[WHOLE ? 0 : j] < lim)
                __builtin_amdgcn_global_load_lds((global_void *)(base + goff[j]),
                                                 (lds_void *)slot, 16, 0, 0);
            else
                *reinterpret_cast<vec *>(slot + lane * VW) = vec{};
        }
    }
};

// Fragments of one step group (VW MFMA steps) for the NB blocks of one side
// of a wavefront's register tile.  Block b's lane l16 stands for tile row
// w0 + block_row<R>(b, l16), as in WaveTile.
template <typename T, int MODE, int NB, int R, int ROWS, int KT>
struct DirectFrag {
    static constexpr int VW = Traits<T>::VW;
    typedef typename Traits<T>::vec vec;
    typedef RVec<T, R> RV;
    static constexpr bool kKV = MODE == kGatherKVec;
    static constexpr bool kKS = MODE == kGatherKVecStrided;
    static constexpr bool kRV = MODE == kGatherRowVec;
    static constexpr int CPR = KT / VW;
    static constexpr int kReads = kKV ? NB : kKS ? VW * NB : VW * (NB / R);   // LDS reads per group
    // k-vector: one piece per block (VW positions of its row); strided
    // k-vector: one element per block and step; row-vector: one read of R
    // rows per block group and step
    vec kv[kKV ? NB : 1];
    T sv[kKS ? VW : 1][kKS ? NB : 1];
    typename RV::type rv[kRV ? VW : 1][kRV ? NB / R : 1];

    __device__ __forceinline__ void read(const T *tile, int w0, int l16, int g, int grp, int es = 1)
    {
        if constexpr (kKS) {
            // position kk = u + es (VW q + e) is element e of piece u nq + q
            // (es is a power of two).  The lanes of one read take the same
            // piece of rows R apart, so the permutation spreads them over
            // the banks as for the k-vector reads, and neighbouring lane
            // groups take neighbouring elements or pieces.
            const int nq = CPR / es, sh = __builtin_ctz(es);
#pragma unroll
            for (int s4 = 0; s4 < VW; ++s4) {
                const int kk = 4 * VW * grp + VW * g + s4;
                const int v = kk >> sh, c = (kk & (es - 1)) * nq + v / VW;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int r = w0 + block_row<R>(b, l16);
                    sv[s4][b] = tile[r * KT + VW * kvec_col<CPR, R>(r, c) + v % VW];
                }
            }
            return;
        }
        if constexpr (kKV) {
            const int q = 4 * grp + g;   // piece of positions kp(VW grp .. VW grp + VW - 1, g)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int r = w0 + block_row<R>(b, l16);
                kv[b] = *reinterpret_cast<const vec *>(tile + r * KT + VW * kvec_col<CPR, R>(r, q));
            }
        } else {
#pragma unroll
            for (int s4 = 0; s4 < VW; ++s4) {
                const int k = 4 * VW * grp + VW * g + s4;
#pragma unroll
                for (int gi = 0; gi < NB / R; ++gi)
                    rv[s4][gi] = *reinterpret_cast<const typename RV::type *>(
                        tile + k * ROWS + w0 + gi * 16 * R + R * l16);
            }
        }
    }
    // the value block b supplies in step s4 of the group
    __device__ __forceinline__ T at(int b, int s4) const
    {
        if constexpr (kKV) return kv[b][s4];
        else if constexpr (kKS) return sv[s4][b];
        else return RV::at(rv[s4][b / R], b % R);
    }
};

// Origins of the K boxes, taken in order (every box whole): the block along
// index kj advances by one; when it wraps, the next contracted index
// advances; only when that one wraps too is the origin decomposed afresh
// (box_origin).  The state is the same on every lane and is kept in scalar
// registers (as vector registers it cost the K loop 3% on the 4096^3-shaped
// fp32 contraction).
struct DirectWalk {
    int64_t ox, oy;     // origin of box `next` in X and Y
    int64_t bx, by;     // step of one block along index kj
    int64_t sx1, sy1;   // strides of index kj + 1
    uint32_t next;
    int blk, c1, nblk, e1, ek, tj;

    __device__ __forceinline__ void init(const KDesc &d, uint32_t s0)
    {
        const KDim &kj = d.k()[d.kj];
        nblk = d.nblk > 0 ? d.nblk : 1;
        ek = kj.ext;
        tj = d.tj;
        bx = (int64_t)d.tj * kj.s0;
        by = (int64_t)d.tj * kj.s1;
        const bool later = d.kj + 1 < d.nk;
        e1 = later ? d.k()[d.kj + 1].ext : 0;
        sx1 = later ? d.k()[d.kj + 1].s0 : 0;
        sy1 = later ? d.k()[d.kj + 1].s1 : 0;
        next = s0;
        uint32_t rest = quotient(s0, nblk, d.nblkInv);
        blk = (int)(s0 - rest * (uint32_t)nblk);
        c1 = later ? (int)digit(rest, d.k()[d.kj + 1]) : 0;
        box_origin(d, s0, ox, oy);
    }
    // origin of box `next` and its valid positions along index kj; then step
    // to the box after it
    __device__ __forceinline__ int take(const KDesc &d, int64_t &x, int64_t &y)
    {
        x = ox;
        y = oy;
        const int lim = ek - blk * tj;
        ++next;
        if (++blk < nblk) {
            ox += bx;
            oy += by;
        } else if (++c1 < e1) {
            blk = 0;
            ox += sx1 - (int64_t)(nblk - 1) * bx;
            oy += sy1 - (int64_t)(nblk - 1) * by;
        } else {
            blk = 0;
            c1 = 0;
            box_origin(d, next, ox, oy);
        }
        blk = uniform(blk);
        c1 = uniform(c1);
        ox = uniform(ox);
        oy = uniform(oy);
        return lim;
    }
};

// One workgroup of the direct-load kernel: boxes [s0, s0 + nsteps) of tile
// `tile`, stored with alpha / beta, or (SLICED) left as a partial tile in `W`.
template <typename T, int MT, int NT, int KT, int WM, int WN, int RX, int RY, int XMODE,
          int YMODE, bool WHOLE, bool SLICED>
__device__ __forceinline__ void direct_tile(const KDesc &d, const T *__restrict__ X,
                                            const T *__restrict__ Y, T *__restrict__ C,
                                            const T alpha, const T beta, int tile, uint32_t s0,
                                            uint32_t nsteps, T *__restrict__ W)
{
    constexpr int NTH = WM * WN * 64;
    constexpr int VW = Traits<T>::VW;
    constexpr int NG = KT / (4 * VW);   // step groups per box
    static_assert(KT % (4 * VW) == 0, "whole step groups");
    typedef WaveTile<T, MT, NT, KT, WM, WN, RX, RY> WT;
    typedef DirectOperand<T, MT, KT, XMODE, NTH, WHOLE, RX> OX;
    typedef DirectOperand<T, NT, KT, YMODE, NTH, WHOLE, RY> OY;
    typedef DirectFrag<T, XMODE, WT::RB, RX, MT, KT> FX;
    typedef DirectFrag<T, YMODE, WT::CB, RY, NT, KT> FY;
    constexpr int STAGE = (MT + NT) * KT;

    // the two box buffers: dynamic LDS of 2 * STAGE elements (the compiler
    // then does not wait for the loads in flight into one buffer before
    // reading the other)
    extern __shared__ __attribute__((aligned(16))) char dyn_lds[];
    T *panels = reinterpret_cast<T *>(dyn_lds);
    __shared__ int rowX[MT], rowY[NT], offCx[MT], offCy[NT];
    __shared__ int kX[KT], kY[KT], kco[KT];

    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    touch_arguments();
    const int ntiles = d.tilesX * d.tilesY;
    box_tables<KT, NTH>(d, tid, kX, kY, kco);
    WT w;
    w.init(tid);
    int tx, ty;
    tile_of_block(d, tile, ntiles, tx, ty);
    const TileBase tb = tile_base<MT, NT>(d, tx, ty);
    tile_tables<MT, NT, NTH>(d, tx, ty, tb, tid, rowX, offCx, rowY, offCy);
    const T *Xt = X + tb.x;
    const T *Yt = Y + tb.y;
    T *Ct = C + (tb.cx + tb.cy);
    __syncthreads();

    OX ox;
    OY oy;
    const int es = YMODE == kGatherKVecStrided ? d.yes : 1;
    ox.setup(tid, rowX, kX, kco);
    oy.setup(tid, rowY, kY, kco, es);
    w.zero();
    const int l16 = tid & 15, g = (tid & 63) >> 4;
    const int xw = w.wm * WT::WTM, yw = w.wn * WT::WTN;

    DirectWalk walk;
    if (nsteps > 0) walk.init(d, s0);
    auto issue = [&](int buf) {   // the boxes in order: s0, s0 + 1, ...
        int64_t bx, by;
        const int lim = walk.take(d, bx, by);
        T *st = panels + buf * STAGE;
        ox.issue(Xt + bx, st, wave, lim);
        oy.issue(Yt + by, st + MT * KT, wave, lim);
    };
    auto read = [&](FX (&fx)[NG], FY (&fy)[NG], int buf) {
        const T *st = panels + buf * STAGE;
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            fx[grp].read(st, xw, l16, g, grp);
            fy[grp].read(st + MT * KT, yw, l16, g, grp, es);
        }
    };
    auto mma = [&](const FX &fx, const FY &fy) {
#pragma unroll
        for (int s4 = 0; s4 < VW; ++s4)
#pragma unroll
            for (int a = 0; a < WT::RB; ++a)
#pragma unroll
                for (int b = 0; b < WT::CB; ++b)
                    w.acc[a][b] = mfma16x16x4(fx.at(a, s4), fy.at(b, s4), w.acc[a][b]);
    };
    // s_barrier with no fence: a workgroup-scope release would wait for the
    // loads in flight into the other buffer (they count as LDS writes)
    auto barrier = []() { asm volatile("s_barrier" ::: "memory"); };
    constexpr int LOADS = OX::J + OY::J;   // load instructions per box and thread
    // s_waitcnt: vmcnt n (gfx9 encoding: low bits 3:0, high bits 15:14),
    // expcnt and lgkmcnt untouched / lgkmcnt 0
    // (lgkmcnt 0 also covers the zeros written in place of pieces outside)
    constexpr int kVmBox = (LOADS & 15) | ((LOADS >> 4) << 14) | (7 << 4);
    constexpr int kVmLgk0 = 7 << 4;
    static_assert(LOADS < 64, "vmcnt range");

    if (nsteps > 0) {
        FX fx[NG];
        FY fy[NG];
        issue(0);
        if (nsteps > 1) {
            issue(1);
            // box 0's loads; box 1's may stay in flight when each box is known
            // to issue all of its loads (a wavefront skips the loads of
            // pieces that are all outside, so the count is not known otherwise)
            __builtin_amdgcn_s_waitcnt(WHOLE ? kVmBox : kVmLgk0);
        } else {
            __builtin_amdgcn_s_waitcnt(kVmLgk0);
        }
        barrier();
        read(fx, fy, 0);
        for (uint32_t s = 0; s + 1 < nsteps; ++s) {
#pragma unroll
            for (int grp = 0; grp + 1 < NG; ++grp) mma(fx[grp], fy[grp]);
            __builtin_amdgcn_s_waitcnt(kVmLgk0);   // box s + 1 loaded, box s read
            barrier();
            if (s + 2 < nsteps) issue((int)(s & 1));   // box s + 2
            FX gx[NG];
            FY gy[NG];
            read(gx, gy, (int)((s + 1) & 1));
            mma(fx[NG - 1], fy[NG - 1]);
            // one fragment read after every few MFMAs of the last group
            constexpr int NREAD = NG * (FX::kReads + FY::kReads);
            constexpr int NMFMA = VW * WT::RB * WT::CB;
#pragma unroll
            for (int r = 0; r < NREAD; ++r) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, NMFMA / NREAD > 0 ? NMFMA / NREAD : 1,
                                                     0);
            }
#pragma unroll
            for (int grp = 0; grp < NG; ++grp) {
                fx[grp] = gx[grp];
                fy[grp] = gy[grp];
            }
        }
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) mma(fx[grp], fy[grp]);
    }
    if constexpr (SLICED) {
#pragma unroll
        for (int a = 0; a < WT::RB; ++a)
#pragma unroll
            for (int b = 0; b < WT::CB; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    W[(size_t)(((a * WT::CB + b) * 4 + r) * NTH + tid)] = w.acc[a][b][r];
    } else {
        w.template unpack<1>(Ct, offCx, offCy, alpha, beta, d.cvec);
    }
}

template <typename T, int MT, int NT, int KT, int WM, int WN, int RX, int RY, int XMODE,
          int YMODE, bool WHOLE>
__global__ void __launch_bounds__(WM *WN * 64) __attribute__((amdgpu_waves_per_eu(2)))
gett_direct_kernel(const KDesc d, const T *__restrict__ X, const T *__restrict__ Y,
                   T *__restrict__ C, const T alpha, const T beta)
{
    direct_tile<T, MT, NT, KT, WM, WN, RX, RY, XMODE, YMODE, WHOLE, false>(
        d, X, Y, C, alpha, beta, d.tile0 + (int)blockIdx.x, 0, (uint32_t)d.nsteps, nullptr);
}

// K slices on the direct-load kernel: workgroup b computes slice b / tiles of
// tile b % tiles into slot b of the workspace (the slots of the macro-kernel's
// K slices), and gett_sum_slices_kernel adds a tile's slots in slice order.
// Bound by the MFMAs: a C of 384 x 376 over 144384 is 9 tiles of 128 x 128
// against 72 tiles of 32 x 64 (64 slices), the largest for which the last
// workgroup of a tile can sum its slots in turn without dominating: 431 us on
// those, 336 here in 56 slices, which fill the CUs twice, 342 in 113, whose
// sums are as short as those of the small tiles.
// Consecutive workgroups of one XCD share a slice's panels in its L2.
template <typename T, int MT, int NT, int KT, int WM, int WN, int RX, int RY, int XMODE,
          int YMODE, bool WHOLE>
__global__ void __launch_bounds__(WM *WN * 64) __attribute__((amdgpu_waves_per_eu(2)))
gett_direct_slice_kernel(const KDesc d, const T *__restrict__ X, const T *__restrict__ Y,
                         T *__restrict__ W)
{
    const int ntiles = d.tilesX * d.tilesY, n = ntiles * d.kslices, full = n & ~7;
    const int bid = (int)blockIdx.x;
    const int b = bid < full ? (bid & 7) * (full >> 3) + (bid >> 3) : bid;
    const int slice = b / ntiles, u = b - slice * ntiles;
    // nsteps < 2^31 and kslices < 2^31 / threads: the products need 64 bits
    const uint32_t s0 = (uint32_t)((uint64_t)d.nsteps * (uint32_t)slice / (uint32_t)d.kslices);
    const uint32_t s1 = (uint32_t)((uint64_t)d.nsteps * (uint32_t)(slice + 1) / (uint32_t)d.kslices);
    direct_tile<T, MT, NT, KT, WM, WN, RX, RY, XMODE, YMODE, WHOLE, true>(
        d, X, Y, nullptr, T(0), T(0), u, s0, s1 - s0, W + (size_t)b * (MT * NT));
}

// C <- alpha * (the sum of a tile's slots, in slice order) + beta * C.  One
// workgroup per MFMA block position (a, b) of the register tile, so that a
// tile's slots are read by 16 workgroups at once; eight slots in flight per
// thread, which are added up before they join the sum (P / 8 + 8 additions in a
// row instead of P).  Bound by the slots' stream from L2 and the Infinity Cache.
template <typename T, int MT, int NT, int KT, int WM, int WN, int RX, int RY>
__global__ void __launch_bounds__(WM *WN * 64)
gett_sum_slices_kernel(const KDesc d, const T *__restrict__ W, T *__restrict__ C, const T alpha,
                       const T beta)
{
    constexpr int NTH = WM * WN * 64;
    constexpr int kFlight = 8;
    typedef WaveTile<T, MT, NT, KT, WM, WN, RX, RY> WT;
    const int ntiles = d.tilesX * d.tilesY;
    const int u = (int)blockIdx.x / (WT::RB * WT::CB);
    const int blk = (int)blockIdx.x - u * (WT::RB * WT::CB);   // a * CB + b
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const T *slot = W + (size_t)u * (MT * NT) + (size_t)blk * 4 * NTH + tid;
    const size_t step = (size_t)ntiles * (MT * NT);
    T sum[4];
    for (int p0 = 0; p0 < d.kslices; p0 += kFlight) {
        T v[kFlight][4];
#pragma unroll
        for (int q = 0; q < kFlight; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                v[q][r] = p0 + q < d.kslices ? slot[(size_t)(p0 + q) * step + r * NTH] : T(0);
#pragma unroll
        for (int q = 1; q < kFlight; ++q)
            if (p0 + q < d.kslices) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[0][r] += v[q][r];
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] = p0 == 0 ? v[0][r] : sum[r] + v[0][r];
    }
    int tx, ty;
    tile_of_block(d, u, ntiles, tx, ty);
    auto offset = [](uint32_t v, int n, const KDim *set) {
        int64_t o = 0;
        for (int i = 0; i < n; ++i) o += (int64_t)digit(v, set[i]) * set[i].s1;
        return o;
    };
    const int col = (wave / WM) * WT::WTN + block_row<RY>(blk % WT::CB, lane & 15);
    const uint32_t y = (uint32_t)(ty * NT + col);
    if ((int64_t)y >= d.sizeY) return;
    const int64_t oy = offset(y, d.ny, d.y());
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = (wave % WM) * WT::WTM +
                        block_row<RX>(blk / WT::CB, Traits<T>::mrow(lane >> 4, r));
        const uint32_t x = (uint32_t)(tx * MT + row);
        if ((int64_t)x >= d.sizeX) continue;
        T *c = C + (oy + offset(x, d.nx, d.x()));
        *c = beta != T(0) ? alpha * sum[r] + beta * *c : alpha * sum[r];
    }
}

// ---------------------------------------------------------------------------
// The direct-load kernel for operands that cannot be gathered in 16-byte
// vectors (odd extents or strides, bases off the 16-byte grid): every element
// is copied into LDS by a load of its own (global_load_lds_dword: lane i of
// one instruction fills bytes [4 i, 4 i + 4) after the wave's LDS base).  The
// LDS images are those of the vector copies, so the fragment reads, the MFMAs
// and the pipeline are the same; four times the load instructions, but nothing
// staged in registers and no alignment to ask for.
//
// Since any element may go to any place, the boxes need not follow the
// indices: box s is positions [s KT, (s + 1) KT) of the linearised contracted
// set, whose offsets are decoded into a small LDS table two boxes ahead.  Only
// the last box can be partial (an extent of 23 in a box of 32 idled 28% of
// the MFMAs).
//
// Bound by the MFMAs on large contractions: 192 load instructions per box of
// a 128 x 256 tile against 8192 cycles of MFMAs per SIMD.
template <typename T, int ROWS, int KT, bool KF, int NTH, int R>
struct ElementOperand {
    static_assert(sizeof(T) == 4, "one dword per element");
    static constexpr int VW = Traits<T>::VW;
    static constexpr int NW = NTH / 64;
    static constexpr int CPR = KT / VW;
    static constexpr int J = ROWS * KT / NTH;   // elements per thread
    // KF: lanes along k, [row][k] with the pieces of a row permuted as for
    // the k-vector copy.  A thread's rows are NTH / KT apart, so its position
    // in the row repeats every P elements.
    static constexpr int P = KF ? (CPR * R * KT / NTH > 1 ? CPR * R * KT / NTH : 1) : 1;
    static_assert(!KF || (NTH % KT == 0 && (NTH / KT) % R == 0 && J % P == 0), "rows per round");
    // otherwise lanes along the rows, [k][row]: one row per thread, one
    // position per wave and element
    static_assert(KF || (NTH % ROWS == 0 && ROWS % 64 == 0 && KT <= 64), "one row per thread");

    uint32_t row[KF ? J : 1];   // operand offset of the element's row
    int kk[P];                  // its box position
    int lane, wave;

    // rowoff: LDS table of operand offsets per tile row; rows outside the
    // tensor load the tile's first row, and nothing reads their results
    __device__ __forceinline__ void setup(int tid, int w, const int *rowoff)
    {
        lane = tid & 63;
        wave = w;
        if constexpr (KF) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int p = (j * NW + w) * 64 + lane, r = p / KT, c = p % KT;
                row[j] = (uint32_t)max(rowoff[r], 0);
                if (j < P) kk[j] = VW * kvec_piece<CPR, R>(r, c / VW) + c % VW;
            }
        } else {
            row[0] = (uint32_t)max(rowoff[tid % ROWS], 0);
            kk[0] = 0;
        }
    }

    // copy this thread's elements of the box whose positions have the offsets
    // `koff` (LDS; -1 past the last position, looked for when CHECK) into `dst`
    template <bool CHECK>
    __device__ __forceinline__ void issue(const T *base, T *dst, const int *koff) const
    {
        int ko[P];
#pragma unroll
        for (int i = 0; i < P; ++i) ko[i] = koff[KF ? kk[i] : lane & (KT - 1)];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            T *slot = dst + (j * NW + wave) * 64;
            int k;
            if constexpr (KF) k = ko[j % P];
            else k = __builtin_amdgcn_readlane(ko[0], (j * NW + wave) * 64 / ROWS);
            if (CHECK && k < 0)
                slot[lane] = T(0);
            else
                __builtin_amdgcn_global_load_lds(
                    (global_void *)(base + (row[KF ? j : 0] + (uint32_t)k)), (lds_void *)slot, 4, 0,
                    0);
        }
    }
};

template <typename T, int MT, int NT, int KT, int WM, int WN, int RX, int RY, bool XKF, bool YKF>
__global__ void __launch_bounds__(WM *WN * 64) __attribute__((amdgpu_waves_per_eu(2)))
gett_element_kernel(const KDesc d, const T *__restrict__ X, const T *__restrict__ Y,
                    T *__restrict__ C, const T alpha, const T beta)
{
    constexpr int NTH = WM * WN * 64;
    constexpr int VW = Traits<T>::VW;
    constexpr int NG = KT / (4 * VW);   // step groups per box
    typedef WaveTile<T, MT, NT, KT, WM, WN, RX, RY> WT;
    typedef ElementOperand<T, MT, KT, XKF, NTH, RX> OX;
    typedef ElementOperand<T, NT, KT, YKF, NTH, RY> OY;
    typedef DirectFrag<T, XKF ? kGatherKVec : kGatherRowVec, WT::RB, RX, MT, KT> FX;
    typedef DirectFrag<T, YKF ? kGatherKVec : kGatherRowVec, WT::CB, RY, NT, KT> FY;
    constexpr int STAGE = (MT + NT) * KT;

    extern __shared__ __attribute__((aligned(16))) char dyn_lds[];
    T *panels = reinterpret_cast<T *>(dyn_lds);
    __shared__ int rowX[MT], rowY[NT], offCx[MT], offCy[NT];
    constexpr int kAhead = 4;   // boxes whose positions are decoded at a time
    __shared__ int kX[2 * kAhead][KT], kY[2 * kAhead][KT];
    static_assert(kAhead * KT <= NTH, "one position per thread");

    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    touch_arguments();
    const int ntiles = d.tilesX * d.tilesY;
    const int nbox = (d.linK + KT - 1) / KT;
    // offsets of position t of box s into its table set
    auto positions = [&](int s, int t) {
        uint32_t k = (uint32_t)(s * KT + t);
        const bool in = k < (uint32_t)d.linK;
        uint32_t ox = 0, oy = 0;
        for (int i = 0; i < d.nk; ++i) {
            const KDim &ki = d.k()[i];
            const uint32_t id = digit(k, ki);
            ox += id * (uint32_t)ki.s0;
            oy += id * (uint32_t)ki.s1;
        }
        kX[s % (2 * kAhead)][t] = in ? (int)ox : -1;
        kY[s % (2 * kAhead)][t] = in ? (int)oy : -1;
    };
    if (tid < 2 * KT) positions(tid / KT, tid % KT);
    WT w;
    w.init(tid);
    int tx, ty;
    tile_of_block(d, d.tile0 + (int)blockIdx.x, ntiles, tx, ty);
    const TileBase tb = tile_base<MT, NT>(d, tx, ty);
    tile_tables<MT, NT, NTH>(d, tx, ty, tb, tid, rowX, offCx, rowY, offCy);
    const T *Xt = X + tb.x;
    const T *Yt = Y + tb.y;
    __syncthreads();

    OX ox;
    OY oy;
    ox.setup(tid, wave, rowX);
    oy.setup(tid, wave, rowY);
    w.zero();
    const int l16 = tid & 15, g = (tid & 63) >> 4;
    const int xw = w.wm * WT::WTM, yw = w.wn * WT::WTN;
    const int whole = d.linK / KT;   // boxes before this one have KT positions
    auto issue = [&](int s) {
        T *st = panels + (s & 1) * STAGE;
        if (s < whole) {
            ox.template issue<false>(Xt, st, kX[s % (2 * kAhead)]);
            oy.template issue<false>(Yt, st + MT * KT, kY[s % (2 * kAhead)]);
        } else {
            ox.template issue<true>(Xt, st, kX[s % (2 * kAhead)]);
            oy.template issue<true>(Yt, st + MT * KT, kY[s % (2 * kAhead)]);
        }
    };
    auto read = [&](FX (&fx)[NG], FY (&fy)[NG], int buf) {
        const T *st = panels + buf * STAGE;
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            fx[grp].read(st, xw, l16, g, grp);
            fy[grp].read(st + MT * KT, yw, l16, g, grp);
        }
    };
    auto mma = [&](const FX &fx, const FY &fy) {
#pragma unroll
        for (int s4 = 0; s4 < VW; ++s4)
#pragma unroll
            for (int a = 0; a < WT::RB; ++a)
#pragma unroll
                for (int b = 0; b < WT::CB; ++b)
                    w.acc[a][b] = mfma16x16x4(fx.at(a, s4), fy.at(b, s4), w.acc[a][b]);
    };
    auto barrier = []() { asm volatile("s_barrier" ::: "memory"); };
    constexpr int kVmLgk0 = 7 << 4;   // vmcnt 0, lgkmcnt 0

    // The pipeline of gett_direct_kernel.  Every kAhead boxes, before the
    // barrier that the loads of box s + 2 follow, the positions of boxes
    // s + 2 .. s + kAhead + 1 are decoded; the sets they replace were read
    // for boxes up to s + 1 - kAhead, issued at least kAhead barriers ago.
    // (Decoding one box at a time cost 5% of the 4096^3 contraction.)
    if (nbox > 0) {
        FX fx[NG];
        FY fy[NG];
        issue(0);
        if (nbox > 1) issue(1);
        __builtin_amdgcn_s_waitcnt(kVmLgk0);
        barrier();
        read(fx, fy, 0);
        for (int s = 0; s + 1 < nbox; ++s) {
            if (s % kAhead == 0 && tid < kAhead * KT) positions(s + 2 + tid / KT, tid % KT);
#pragma unroll
            for (int grp = 0; grp + 1 < NG; ++grp) mma(fx[grp], fy[grp]);
            __builtin_amdgcn_s_waitcnt(kVmLgk0);   // box s + 1 loaded, box s read
            barrier();
            if (s + 2 < nbox) issue(s + 2);
            FX gx[NG];
            FY gy[NG];
            read(gx, gy, (s + 1) & 1);
            mma(fx[NG - 1], fy[NG - 1]);
            constexpr int NREAD = NG * (FX::kReads + FY::kReads);
            constexpr int NMFMA = VW * WT::RB * WT::CB;
#pragma unroll
            for (int r = 0; r < NREAD; ++r) {
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, NMFMA / NREAD > 0 ? NMFMA / NREAD : 1,
                                                     0);
            }
#pragma unroll
            for (int grp = 0; grp < NG; ++grp) {
                fx[grp] = gx[grp];
                fy[grp] = gy[grp];
            }
        }
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) mma(fx[grp], fy[grp]);
    }
    w.template unpack<1>(C + (tb.cx + tb.cy), offCx, offCy, alpha, beta, d.cvec);
}

// Persistent direct-load kernel for plans whose contracted set is one K box.
// Workgroups walk tiles t = tile0 + blockIdx.x, + gridDim.x, ...; tile t's box
// sits in LDS buffer t mod 2 (per workgroup).  Per tile:
//   LDS reads of tile t's fragments; offset tables of the next tile (second
//     table set); barrier;
//   the copy of the next tile's box into the other buffer;
//   MFMAs of tile t; its C stores (unpack);
//   wait for this wavefront's copy; barrier.
// The copy is issued before the C stores of tile t, so it does not queue
// behind them (a CU serves its vector memory instructions in order), and the
// wait for it leaves those stores in flight: vmcnt counts in issue order and
// every tile issues at least kStores vector memory instructions after its
// copy when every piece is inside the tensors (WHOLE); otherwise the wait
// is for everything (vmcnt 0).
template <typename T, int MT, int NT, int KT, int WM, int WN, int RX, int RY, int XMODE, int YMODE,
          bool WHOLE>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(2))) void
gett_direct_stream_kernel(const KDesc d, const T *__restrict__ X, const T *__restrict__ Y,
                          T *__restrict__ C, const T alpha, const T beta)
{
    constexpr int NTH = WM * WN * 64;
    constexpr int VW = Traits<T>::VW;
    constexpr int NG = KT / (4 * VW);   // step groups per box
    static_assert(KT % (4 * VW) == 0, "whole step groups");
    typedef WaveTile<T, MT, NT, KT, WM, WN, RX, RY> WT;
    typedef DirectOperand<T, MT, KT, XMODE, NTH, WHOLE, RX> OX;
    typedef DirectOperand<T, NT, KT, YMODE, NTH, WHOLE, RY> OY;
    typedef DirectFrag<T, XMODE, WT::RB, RX, MT, KT> FX;
    typedef DirectFrag<T, YMODE, WT::CB, RY, NT, KT> FY;
    constexpr int STAGE = (MT + NT) * KT;
    // vector memory instructions each wavefront issues after a copy: the C
    // stores of one tile, vectors or single elements (C loads with beta != 0
    // only add to them)
    constexpr int kStores = (WT::RB / RX) * WT::NR * (WT::kVecC ? WT::CGV : WT::CB);
    constexpr int kAfter = kStores < 63 ? kStores : 63;
    // s_waitcnt (gfx9 encoding): vmcnt kAfter / vmcnt 0, lgkmcnt 0 / lgkmcnt
    // 0 alone (vmcnt 63), expcnt untouched
    constexpr int kVmAfter = (kAfter & 15) | ((kAfter >> 4) << 14) | (7 << 4) | (15 << 8);
    constexpr int kVmLgk0 = 7 << 4;
    constexpr int kLgk0 = 15 | (3 << 14) | (7 << 4);

    extern __shared__ __attribute__((aligned(16))) char dyn_lds[];
    T *panels = reinterpret_cast<T *>(dyn_lds);
    __shared__ int rowX[2][MT], rowY[2][NT], offCx[2][MT], offCy[2][NT];
    __shared__ int kX[KT], kY[KT], kco[KT];

    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntiles = d.tilesX * d.tilesY;
    box_tables<KT, NTH>(d, tid, kX, kY, kco);
    int64_t bx0, by0;
    const int lim = box_origin(d, 0, bx0, by0);
    WT w;
    w.init(tid);
    const int l16 = tid & 15, g = (tid & 63) >> 4;
    const int xw = w.wm * WT::WTM, yw = w.wn * WT::WTN;
    OX ox;
    OY oy;
    auto barrier = []() { asm volatile("s_barrier" ::: "memory"); };
    // offset tables of tile t into table set `set`; the tile's operand and C bases
    auto prepare = [&](int t, int set, const T *&Xt, const T *&Yt, T *&Ct) {
        int tx, ty;
        tile_of_block(d, t, ntiles, tx, ty);
        const TileBase tb = tile_base<MT, NT>(d, tx, ty);
        tile_tables<MT, NT, NTH>(d, tx, ty, tb, tid, rowX[set], offCx[set], rowY[set], offCy[set]);
        Xt = X + (tb.x + bx0);
        Yt = Y + (tb.y + by0);
        Ct = C + (tb.cx + tb.cy);
    };
    auto issue = [&](int set, const T *Xt, const T *Yt, int buf) {
        ox.setup(tid, rowX[set], kX, kco);
        oy.setup(tid, rowY[set], kY, kco);
        T *st = panels + buf * STAGE;
        ox.issue(Xt, st, wave, lim);
        oy.issue(Yt, st + MT * KT, wave, lim);
    };
    auto mma = [&](const FX &fx, const FY &fy) {
#pragma unroll
        for (int s4 = 0; s4 < VW; ++s4)
#pragma unroll
            for (int a = 0; a < WT::RB; ++a)
#pragma unroll
                for (int b = 0; b < WT::CB; ++b)
                    w.acc[a][b] = mfma16x16x4(fx.at(a, s4), fy.at(b, s4), w.acc[a][b]);
    };

    int t = d.tile0 + (int)blockIdx.x;   // the grid holds no more workgroups than tiles
    const T *Xt, *Yt;
    T *Ct;
    prepare(t, 0, Xt, Yt, Ct);
    __syncthreads();
    issue(0, Xt, Yt, 0);
    __builtin_amdgcn_s_waitcnt(kVmLgk0);
    barrier();
    int cur = 0;
    for (;;) {
        FX fx[NG];
        FY fy[NG];
        const T *st = panels + cur * STAGE;
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) {
            fx[grp].read(st, xw, l16, g, grp);
            fy[grp].read(st + MT * KT, yw, l16, g, grp);
        }
        const int tn = t + (int)gridDim.x;
        const bool more = tn < ntiles;
        const T *Xn = Xt, *Yn = Yt;
        T *Cn = Ct;
        if (more) prepare(tn, cur ^ 1, Xn, Yn, Cn);
        // this tile's fragments are in registers, the next tile's tables complete
        __builtin_amdgcn_s_waitcnt(kLgk0);
        barrier();
        if (more) issue(cur ^ 1, Xn, Yn, cur ^ 1);
        // the copy stays ahead of the stores below in issue order
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        w.zero();
#pragma unroll
        for (int grp = 0; grp < NG; ++grp) mma(fx[grp], fy[grp]);
        w.template unpack<1, WHOLE>(Ct, offCx[cur], offCy[cur], alpha, beta, d.cvec);
        if (!more) break;
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        // the next tile's box has landed (this wavefront's part; the barrier
        // covers the others); this tile's stores may still be in flight
        __builtin_amdgcn_s_waitcnt(WHOLE ? kVmAfter : kVmLgk0);
        barrier();
        t = tn;
        Xt = Xn;
        Yt = Yn;
        Ct = Cn;
        cur ^= 1;
    }
}

}  // namespace gett
