// The screening bounds by line, the certificates of the lean sweep and the rule by which it renews its bounds: plain
// arithmetic, no HIP in here.  drot.hip includes it with DROT_FN set for device code, the CPU tests compile the same lines
// for the host.

// The bounds by line: how far below M the largest t_j of each of the segment's eight 128-byte lines (32 columns) lies, one
// byte per line.  The byte is the number's exponent and three bits of its fraction, cut off (towards 0: M minus the
// decoded number is never below the line's true maximum), over 32 octaves around the size of rho (costs are of order 1):
// from 2^-15 rho, below which it says 0, to 2^17 rho, where it saturates.
DROT_FN int line_code_base(float rho) { return ((__builtin_bit_cast(int, rho) >> 23) - 15) * 8; }
DROT_FN unsigned line_code(float below, int base) {
  const int code = (__builtin_bit_cast(int, below) >> 20) - base;
  return (unsigned)(code < 0 ? 0 : code > 255 ? 255 : code);
}
DROT_FN float line_decode(unsigned code, int base) {
  return code == 0 ? 0.f : __builtin_bit_cast(float, ((int)code + base) << 20);
}

// The two certificates of the lean sweep.  A segment: max(M + drift of column j*, M2 + largest drift) + phi_i; one of its
// lines: M minus the line's byte (below: decoded) + the line's drift + phi_i.  (With the drift of the line of j* in place
// of its own, three times as many lines are read after a hundred sweeps.)  mag: magnitude of the largest drift plus that of
// varphi.  Margin 16 half units in the last place (2^-20) of what stands beside M.  With u half a unit, a number t_j on
// record is off by u |t_j|, a drift d_j by u |d_j|, their sum and the sum with phi_i by u of what they come to, and the
// sweep adds phi_i to varphi_j within u of that.  Where the true sum is close to zero, |t_j| <= |d_j| + |phi_i|, and all of
// it is at most u (2 |d_j| + 3 |phi_i| + |varphi_j|); where |t_j| is more than twice |d_j| + |phi_i|, the sign is that of
// t_j.  Of column j* the drift can be anything: its magnitude is drift1's own.  Any other column lies below M2 + drift by
// at least what its drift is below the largest one, which covers u of it.  (The line's byte: M counts as well.)
constexpr float kLeanEps = 9.53674316e-7f;  // 2^-20
DROT_FN bool certified_segment(float m1, float m2, float drift1, float drift, float mag, float ph) {
  const float bound = fmaxf(m1 + drift1, m2 + drift) + ph;
  return bound + kLeanEps * (fabsf(ph) + mag + fabsf(drift1)) <= 0.f;  // (-inf where every pair of the segment is forbidden)
}
DROT_FN bool certified_line(float m1, float below, float drift, float mag, float ph) {
  if (m1 == -INFINITY) return true;
  const float bound = ((m1 - below) + drift) + ph;
  return bound + kLeanEps * (fabsf(m1) + fabsf(ph) + mag) <= 0.f;
}

// The active entries (drot_active.h): may a zero entry come to hold something while phi_i and varphi_j together rise by less than tau?
// t: varphi_j - rho C_ij as the sweep's own fmaf gives it.  A line of entries: its bound, which was of some earlier varphi's t and is
// off by u of itself, plus the rise of varphi since; mag: the rise's magnitude plus the largest of varphi in the line.  The margin, 16 u of every term,
// covers u |t| of t, 2 u of the sums here, and u (|varphi_j| + |phi_i|) of the sum that the sweep forms of phi_i and varphi_j before it
// takes off rho C_ij (t cancels, varphi_j does not); what that sum is off by in a later sweep is part of the rise (active_rise).
DROT_FN bool active_entry(float t, float vp, float ph, float tau) {
  return (t + ph) + tau > -kLeanEps * (((fabsf(t) + fabsf(vp)) + fabsf(ph)) + tau);
}
DROT_FN bool active_line(float bound, float rise, float mag, float ph, float tau) {
  return ((bound + rise) + ph) + tau > -kLeanEps * (((fabsf(bound) + mag) + fabsf(ph)) + tau);
}
// How far a number of phi or varphi has risen, and two rises, or a rise and one that is known already, together.
DROT_FN float active_rise(float now, float from) { return (now - from) + kLeanEps * (fabsf(now) + fabsf(from)); }
DROT_FN float active_rises(float a, float b) { return (a + b) + kLeanEps * (fabsf(a) + fabsf(b)); }

// When the lean sweep renews its bounds, the classic rent-or-buy rule: reading lines in vain (zero before and zero after:
// the bounds failed to certify them) is the rent, renewing the bounds (all of C once) the purchase.  Renew when the rent
// paid since the last renewal has reached the price.  That stays within a factor 2 of the best schedule in hindsight,
// whatever the drift of varphi does, and needs no model of it.
struct Renewal {
  int renew;  // the next lean sweep renews the bounds
  int since;  // lean sweeps since the last renewal
  int paid;   // lines read in vain since
};
// After a lean sweep that read `waste` lines in vain, or, where it was asked to, has renewed the bounds.
DROT_FN Renewal after_lean_sweep(Renewal R, int waste, int price, int max_since) {
  if (R.renew) return Renewal{0, 0, 0};
  constexpr int kMost = 1000000000;  // (a sum that stays in range whatever the size)
  R.since += 1;
  R.paid += waste < kMost - R.paid ? waste : kMost - R.paid;
  R.renew = R.paid >= price || R.since >= max_since;
  return R;
}
