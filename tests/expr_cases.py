"""Long user kernels for the tests of generated kernels."""
PIXELS = ["a[%d, %d]" % (x, y) for y in range(-2, 3) for x in range(-2, 3)]


def long_expressions(terms):
    """Sums of `terms` window pixels, halved, saturated and under abs()."""
    s = "(" + " + ".join(PIXELS[:terms]) + ")"
    return ["abs(%s - 700) / 2" % s, "abs(%s) / 2 - %s" % (s, PIXELS[24]), "abs(%s - 300) / 4" % s,
            "abs(abs(%s - 300) - 200)" % s]
