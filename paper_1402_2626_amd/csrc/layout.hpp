// Device-side layout of a packed system.  Shared by the host packer and the
// kernels; plain C++ so the packer builds without HIP.
//
// A polynomial's monomials are cut into CHUNKS.  A chunk is processed by one
// workgroup in one pass: every monomial of the chunk gets a group of `s`
// consecutive lanes (s a power of two, at most one wavefront), lane q of the
// group handles the SEGMENT of the monomial's occurrences q, q + s, q + 2s, ...
// (at most `seg` of them; occurrences in variable order), and each partial
// derivative is written to its own LDS SLOT.
// Slots are numbered so that the contributions to one Jacobian column are
// contiguous: column c owns slots colptr[c] .. colptr[c+1]-1.  This
// owner-computes order is fixed at load time, so results are bitwise
// reproducible.  Every lane walks all `seg` records of the chunk: positions
// past the end of its segment hold a neutral record (variable n, which the
// kernels read as the constant 1, exponent 1, and the chunk's dummy slot
// `nslots`, which no column owns).  The monomial values (the terms of F) do
// not go through slots.
#pragma once
#include <cstdint>

namespace pe {

// one occurrence of a variable in a monomial, stored lane-major per chunk:
// record i of lane lam of chunk ch is at occ[ch.occ_base + i * ch.width + lam]
struct alignas(8) OccRec {
  uint16_t var;   // variable index
  uint16_t exp;   // exponent (>= 1)
  uint16_t slot;  // LDS slot of this partial derivative within the chunk (nslots: dummy)
  uint16_t pad;
};

struct ChunkDesc {
  uint32_t occ_base;     // first OccRec of the chunk
  uint32_t mon_base;     // first monomial (packed order) of the chunk
  uint32_t colptr_base;  // first colptr entry of the chunk (n + 1 entries)
  uint32_t poly;         // polynomial the chunk belongs to
  uint16_t count;        // monomials in the chunk
  uint16_t nslots;       // slots used; slot nslots is the dummy
  uint16_t width;        // lanes used = count * s (the OccRec row stride)
  uint8_t s;             // lanes per monomial (power of two, <= 64)
  uint8_t seg;           // records per lane = ceil(kmax / s)
};

// per-monomial metadata (packed order): the number of variables k
inline uint32_t mon_meta(uint32_t k) { return k; }

constexpr int kRealLevel = 8;  // flag of the level code for real numbers
constexpr uint32_t kNoOcc = 0xffffffffu;  // input occurrence index of a neutral record
constexpr int kRowDesc = 4;      // first chunk descriptors of each row, stored by row
constexpr int kMaxVars = 65535;
constexpr int kMaxSeg = 16;      // largest segment any kernel variant handles
constexpr int kMaxWave = 64;     // lanes per wavefront on gfx950
constexpr int kMaxMonomialVars = kMaxWave * kMaxSeg;  // 1024

// ------------------------------------------------------------------ value layout
//
// A second packing of the same system for the evaluation through monomial
// values (value_kernels.hpp): the product phase takes UNITS of one wavefront,
// the column phase the rows' occurrences by COLUMN.
//
// A unit is up to 64 / s monomials, s lanes each (a power of two); lane l's
// record i is rec[base + 64 i + l], the index (exp - 1) (n + 1) + var of the
// factor in the table of powers, padded with the neutral record n (variable
// n, the constant 1).  The monomials of a row are in the same
// order as in the chunks (larger first).
struct ValUnit {
  uint32_t base;  // first record
  uint16_t mon;   // first monomial, counted from the block's first
  uint8_t count;  // monomials
  uint8_t lgs;    // log2 of the lanes per monomial
  uint32_t seg;   // records per lane
  uint32_t pad;
};

// A block is a run of a row's units whose monomial values fit in LDS together.
// Its column lists are stored in slices of 64 lanes, Q lanes per column, the
// row's columns in decreasing length (val_perm): entry i of lane l of slice c
// is ell[64 (slice[slice0 + c] + i) + l], monomial (from the block's first) |
// exponent << 16, padded with the dummy monomial `nmon` (value 0) and
// exponent 0; the slice ends at slice[slice0 + c + 1].
struct ValBlock {
  uint32_t unit0, unit1;
  uint32_t mon0;      // first monomial (packed order)
  uint32_t nmon;
  uint32_t slice0;
  uint32_t pad;
};

}  // namespace pe
